// First-hit traversal of sparse voxel octrees with transformed subtrees, for
// gfx950 (wave64; no matrix cores: the work is dependent 8-byte gathers).
//
// Per ray (one lane each):
//   1. map the world ray into a frame's grid coordinates (paper Eq. 2-3 with
//      the scale folded into the affine map, Sec. 3.2); t is not rescaled;
//   2. mirror axes with a negative direction so every component is positive;
//      a plane crossing is then t(v) = v * invd + bias, one FMA, evaluated by
//      the same formula for every cell sharing that plane;
//   3. walk the frame's octree front to back, top-down (the role of the
//      parametric traversal in the paper, Sec. 5): integer cell corners, a
//      per-level LDS stack of (child start, mask), and an exit by the highest
//      changed coordinate bit, so popping needs no search (4 bytes per
//      level and lane: a 24-bit child start and an 8-bit mask in one word;
//      5 bytes where a pool needs wider child starts, see kWide);
//   4. at a transformed node whose moved content stays inside its static
//      cell, switch into that node's frame in place (Sec. 3, Fig. 1: the ray,
//      not the model, is transformed) and resume the enclosing walk after it;
//   5. transformed subtrees that leave their static cell are candidates,
//      traced from their own roots in order of root-cell entry and skipped
//      once it lies beyond the best hit (the depth sort of Sec. 4.2): after
//      the walk of the world frame each ray lists the nearest of those that
//      it may enter before its hit, by the bounding-sphere test of Sec. 4.1
//      and the slab entry, up to 16 tested one by one, more through a
//      hierarchy of their world boxes;
//   6. at the hit, recompute its entry t and face from the frame's FP64 map
//      (the walk's FP32 entry t carries an error that grows with the
//      coordinates); write id, slot, t and the normal (entry face, inverse
//      transpose).
//
// Work distribution: a persistent grid.  Each wave keeps 64 rays in flight
// and refills lanes once `refill` of them are idle (64 = whole tiles), from
// a range of `claim` rays it takes at once from one of kQueueParts counters
// (claims interleaved over the counters, each wave starting on its own), so
// that no single address serialises the claims.  Claims visit the 64-ray
// tiles in a stride permutation, so that expensive regions of an image (rays
// grazing a surface) spread over time and over waves instead of reaching a
// few waves back to back.  The last work-group to finish resets the counters
// so the next launch on the stream starts from zero.
//
// Slow tiles first (one-job launches with whole tiles): a launch ends when
// its longest chains of walk steps do, and the same rays traced again (an
// animation under a fixed camera) have their costliest tiles in nearly the
// same places.  Each launch lists the tiles whose longest ray took the most
// advances in its work queue's state (kHot*), and the next launch on the same
// rays deals those tiles to its waves before any regular claim, while the
// regular order skips them; results never depend on the order.
//
// What bounds it: instruction issue while tiles are left (56 % of the VALU
// rate over a whole 1080p terrain launch under a moving camera, 83 % over a 4K
// launch on the 4096^3 terrain), then the longest chains of dependent walk steps; memory only
// through their latency (the 1080p terrain moves 116 MB of rays and hits in
// 127 us).  So the walk is laid out for few instructions per step: one turn of
// its loop advances and then descends (14.4 turns per 64-ray tile where a turn
// that did either took 19.5), node words come ready to push (absolute child
// starts, encoded at upload), and the loop keeps no lane masks.  Together with
// the queue, the candidate listing, the register budgets and the streaming
// hints below: 1080p terrain under moving cameras 221 -> 150 us, the same rays
// again 185 -> 129, 64 instances 398 -> 252, 4K on the 4096^3 terrain 2,159 ->
// 1,482.
#include <hip/hip_runtime.h>

#include <cstring>
#include <mutex>
#include <type_traits>

#include "svo_camera.h"
#include "svo_internal.h"

namespace svo {

namespace {

constexpr uint32_t kNone = 0xFFFFFFFFu;
constexpr uint32_t kStepLimitId = 0xFFFFFFFEu;
enum : uint32_t { M_DONE = 0, M_WALK = 1, M_SELECT = 2 };
enum : uint32_t { EV_NONE = 0, EV_HIT = 1, EV_ENTER = 2, EV_END = 3, EV_LIMIT = 4 };
enum : uint32_t { PEND_RESUME = 1, PEND_ROOT_HIT = 2 };
constexpr uint32_t kUnlisted = ~0u, kListMore = 0x100u;

struct Ray {
    float ox, oy, oz, tmin, dx, dy, dz, tmax;
};

// A ray in one frame's mirrored grid coordinates.
struct FrameRay {
    float ix, iy, iz;   // 1 / |d_a|
    float bx, by, bz;   // t(v) = v * i_a + b_a for the mirrored plane v
    uint32_t flip;      // bit a: d_a < 0 in the frame (axis mirrored)
    uint32_t K;         // frame height
};

__device__ __forceinline__ float min3f(float a, float b, float c) { return fminf(fminf(a, b), c); }

// Reciprocal, square root and reciprocal square root on the hardware units
// (v_rcp_f32, v_sqrt_f32, v_rsq_f32: about 1 ulp) instead of the correctly
// rounded sequences.  Uses: the walk's plane parameters (one reciprocal per
// axis, used for every plane, so the walk stays self-consistent and
// monotone), the inflated bounding-sphere test and normals.  Arguments stay
// in the normal range: rays whose direction is below 2^-100 in every
// component miss (ray_valid), and a frame's clamped components are at least
// 2^-21 of its largest.
__device__ __forceinline__ float rcp_fast(float x) { return __builtin_amdgcn_rcpf(x); }
__device__ __forceinline__ float sqrt_fast(float x) { return __builtin_amdgcn_sqrtf(x); }
__device__ __forceinline__ float rsq_fast(float x) { return __builtin_amdgcn_rsqf(x); }
__device__ __forceinline__ float max3f(float a, float b, float c) { return fmaxf(fmaxf(a, b), c); }

// Map the ray into frame F and clip it to the root cell [0, 2^K)^3 and
// [tmin, tlimit].  Returns false when that interval is empty.  kPrecise:
// the plane parameters take correctly rounded reciprocals (a walk runs on
// them, and the error of every plane crossing it compares includes theirs:
// on the depth-12 terrain this takes the share of rays whose voxel differs
// from the exact one by about a tenth); otherwise the hardware reciprocal
// (entry tests that only order or cull).
template <bool kPrecise>
__device__ __forceinline__ bool frame_setup(const FrameRec& F, const Ray& r, float tlimit, FrameRay& fr, float& t0) {
    const float gx = fmaf(F.m[0], r.ox, fmaf(F.m[1], r.oy, fmaf(F.m[2], r.oz, F.m[3])));
    const float gy = fmaf(F.m[4], r.ox, fmaf(F.m[5], r.oy, fmaf(F.m[6], r.oz, F.m[7])));
    const float gz = fmaf(F.m[8], r.ox, fmaf(F.m[9], r.oy, fmaf(F.m[10], r.oz, F.m[11])));
    float dx = fmaf(F.m[0], r.dx, fmaf(F.m[1], r.dy, F.m[2] * r.dz));
    float dy = fmaf(F.m[4], r.dx, fmaf(F.m[5], r.dy, F.m[6] * r.dz));
    float dz = fmaf(F.m[8], r.dx, fmaf(F.m[9], r.dy, F.m[10] * r.dz));
    const uint32_t K = (F.info >> FR_K_SHIFT) & FR_K_MASK;
    const float N = (float)(1u << K);
    // A zero component would make 0 * inf; a tiny one of the same sign keeps
    // every plane crossing finite and far outside the root cell.
    const float eps = max3f(fabsf(dx), fabsf(dy), fabsf(dz)) * 0x1p-21f;
    if (fabsf(dx) < eps) dx = copysignf(eps, dx);
    if (fabsf(dy) < eps) dy = copysignf(eps, dy);
    if (fabsf(dz) < eps) dz = copysignf(eps, dz);
    fr.flip = (dx < 0.f ? 1u : 0u) | (dy < 0.f ? 2u : 0u) | (dz < 0.f ? 4u : 0u);
    if constexpr (kPrecise) {
        fr.ix = 1.0f / fabsf(dx);
        fr.iy = 1.0f / fabsf(dy);
        fr.iz = 1.0f / fabsf(dz);
    } else {
        fr.ix = rcp_fast(fabsf(dx));
        fr.iy = rcp_fast(fabsf(dy));
        fr.iz = rcp_fast(fabsf(dz));
    }
    fr.bx = -((dx < 0.f) ? (N - gx) : gx) * fr.ix;
    fr.by = -((dy < 0.f) ? (N - gy) : gy) * fr.iy;
    fr.bz = -((dz < 0.f) ? (N - gz) : gz) * fr.iz;
    fr.K = K;
    // root entry: the low mirrored planes are at 0, so t(0) = bias
    float te = max3f(fr.bx, fr.by, fr.bz);
    const float tx = min3f(fmaf(N, fr.ix, fr.bx), fmaf(N, fr.iy, fr.by), fmaf(N, fr.iz, fr.bz));
    if (te < r.tmin) te = r.tmin;
    t0 = te;
    return te <= fminf(tx, tlimit);
}

// Slow-tiles-first state (see kHotHdr): which list is the input, the
// threshold, a list's tiles and its bitmap.  The header stays fixed during a
// launch until its last work-group rewrites it.
__device__ __forceinline__ uint32_t hot_in(const uint32_t* hot) { return hot[0] & 1u; }
__device__ __forceinline__ uint32_t hot_thr(const uint32_t* hot) { return hot[1] ? hot[1] : kHotInitialThreshold; }
__device__ __forceinline__ uint32_t* hot_cnt(uint32_t* hot, uint32_t b, uint32_t s) {
    return hot + kHotCntBase + (b * kHotSub + s) * kHotLine;
}
__device__ __forceinline__ uint32_t* hot_sum(uint32_t* hot, uint32_t s) { return hot + kHotSumBase + s * kHotLine; }
__device__ __forceinline__ uint32_t* hot_max(uint32_t* hot, uint32_t s) { return hot + kHotMaxBase + s * kHotLine; }
__device__ __forceinline__ uint32_t* hot_list(uint32_t* hot, uint32_t b) { return hot + kHotHdr + b * kHotCap; }
__device__ __forceinline__ uint32_t* hot_bits(uint32_t* hot, uint32_t b) {
    return hot + kHotHdr + 2 * kHotCap + b * kHotBitsWords;
}

// The largest of a wave's 64 values, wave-uniform: within each row of 16
// lanes by DPP moves (swap neighbours, swap pairs, mirror the half-rows,
// mirror the rows), then over the four rows by lane reads.  Every lane must
// be active.
__device__ __forceinline__ uint32_t wave_max(uint32_t v) {
    v = max(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0xB1, 0xF, 0xF, false));   // quad_perm 1,0,3,2
    v = max(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x4E, 0xF, 0xF, false));   // quad_perm 2,3,0,1
    v = max(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x141, 0xF, 0xF, false));  // row_half_mirror
    v = max(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x140, 0xF, 0xF, false));  // row_mirror
    const uint32_t r = max(max((uint32_t)__builtin_amdgcn_readlane((int)v, 0), (uint32_t)__builtin_amdgcn_readlane((int)v, 16)),
                           max((uint32_t)__builtin_amdgcn_readlane((int)v, 32), (uint32_t)__builtin_amdgcn_readlane((int)v, 48)));
    return (uint32_t)__builtin_amdgcn_readfirstlane((int)r);
}

// A value the compiler knows nothing about from here on: a branch on it stays
// one branch, where a value known along some path would be threaded into
// copies of the code around it.
__device__ __forceinline__ void opaque(uint32_t& v) { asm("" : "+v"(v)); }

// Wait until this wave's memory operations, atomics without a result among
// them, have completed.
__device__ __forceinline__ void wait_memory() {
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_waitcnt(0);
    asm volatile("" ::: "memory");
}

// The slow-tile state's address from a work-group's LDS header.
__device__ __forceinline__ uint32_t* lds_hot_ptr(const uint32_t* lds_hot) {
    return reinterpret_cast<uint32_t*>((uint64_t)lds_hot[kHotLdsPtr] | ((uint64_t)lds_hot[kHotLdsPtr + 1] << 32));
}
// A wave-uniform value in scalar registers of its own.
__device__ __forceinline__ uint32_t uniform_u32(uint32_t v) { return (uint32_t)__builtin_amdgcn_readfirstlane((int)v); }
template <typename T>
__device__ __forceinline__ T* uniform_ptr(T* p) {
    const uint64_t v = reinterpret_cast<uint64_t>(p);
    return reinterpret_cast<T*>((uint64_t)uniform_u32((uint32_t)v) | ((uint64_t)uniform_u32((uint32_t)(v >> 32)) << 32));
}

// The hit the walk found, checked and measured in FP64.  The walk decides
// in FP32 which cell the ray meets first; its plane crossings carry an
// error that grows with the coordinates (frame map, reciprocal direction,
// rounding at the scale of t), so near an edge or a corner it may take a
// cell the ray passes by, and its entry t is off by that much.  Here the
// cell [p, p + size)^3 (p in frame F's mirrored grid coordinates) is
// intersected with the ray mapped by F's exact map X in FP64 (Eq. 2: the
// frame's ray keeps the world t): per axis the closed slab between the
// cell's two face planes.  Returns whether max(t_near, tmin) <= min(t_far,
// tmax) holds in FP64; then t = max(t_near, tmin) and axis = the entry face
// (the largest t_near, ties to the lowest axis), 3 when the ray starts
// inside the cell (t = tmin).
__device__ __forceinline__ bool exact_hit(const double* X, const Ray& r, const FrameRay& fr, uint32_t px,
                                          uint32_t py, uint32_t pz, uint32_t size, float& t, int& axis) {
    const double N = (double)(1ull << fr.K), S = (double)size;
    double tn = -INFINITY, tf = INFINITY;
    int ea = 3;
    // one axis at a time: a row's four doubles are the only FP64 values live
#pragma unroll 1
    for (int k = 0; k < 3; ++k) {
        const double* row = X + 4 * k;
        const double go = fma(row[0], (double)r.ox, fma(row[1], (double)r.oy, fma(row[2], (double)r.oz, row[3])));
        const double gd = fma(row[0], (double)r.dx, fma(row[1], (double)r.dy, row[2] * (double)r.dz));
        const uint32_t pk = (k == 0) ? px : ((k == 1) ? py : pz);
        const double lo = ((fr.flip >> k) & 1u) ? N - (double)pk - S : (double)pk;
        const double hi = lo + S;
        double a, b;
        if (gd == 0.0) {
            // parallel: the whole line or nothing
            a = (go >= lo && go <= hi) ? -INFINITY : INFINITY;
            b = (go >= lo && go <= hi) ? INFINITY : -INFINITY;
        } else {
            // reciprocal: hardware estimate and two Newton steps (within an
            // ulp or two of 1 / gd; gd is far from the subnormal range)
            double inv = __builtin_amdgcn_rcp(gd);
            inv = fma(inv, fma(-gd, inv, 1.0), inv);
            inv = fma(inv, fma(-gd, inv, 1.0), inv);
            const double t1 = (lo - go) * inv, t2 = (hi - go) * inv;
            a = fmin(t1, t2);
            b = fmax(t1, t2);
        }
        if (a > tn) {
            tn = a;
            ea = k;
        }
        tf = fmin(tf, b);
    }
    double te = tn;
    if (!(te >= (double)r.tmin)) {
        te = (double)r.tmin;
        ea = 3;
    }
    t = (float)te;
    axis = ea;
    return te <= fmin(tf, (double)r.tmax);
}

// Bounding-sphere test of the paper's Sec. 4.1 (Eq. 4), made conservative
// for FP32: false only when the ray segment [tmin, tlimit] certainly misses
// the sphere (its perpendicular distance exceeds the radius, or the sphere
// lies wholly before tmin or after tlimit).  To absorb rounding the radius
// is inflated by a relative 1e-4 (sp.w is its square), and that square by
// 1e-6 of the squared centre distance (about 1e-3 of the distance).  A miss
// costs 13 instructions.
__device__ __forceinline__ bool sphere_may_hit(const float4 sp, const Ray& r, float tlimit) {
    const float lx = sp.x - r.ox, ly = sp.y - r.oy, lz = sp.z - r.oz;
    const float idd = rcp_fast(fmaf(r.dx, r.dx, fmaf(r.dy, r.dy, r.dz * r.dz)));
    const float ll = fmaf(lx, lx, fmaf(ly, ly, lz * lz));
    const float tca = fmaf(lx, r.dx, fmaf(ly, r.dy, lz * r.dz));
    const float tc = tca * idd;                            // t of the closest approach
    const float perp2 = fmaf(-tca, tc, ll * (1.f - 1e-6f)); // squared distance of the line, less the slack
    if (perp2 > sp.w) return false;
    const float half = sqrt_fast(fmaxf(sp.w - perp2, 0.f) * idd);  // half chord, in t
    return (tc - half <= tlimit) && (tc + half >= r.tmin);
}

// A ray's inverse world direction and -origin times it, for box tests; tiny
// components clamped as in frame_setup (so no 0 * inf).
struct BoxRay {
    float ix, iy, iz, nx, ny, nz;
};

__device__ __forceinline__ BoxRay box_ray(const Ray& r) {
    const float eps = max3f(fabsf(r.dx), fabsf(r.dy), fabsf(r.dz)) * 0x1p-21f;
    BoxRay b;
    b.ix = rcp_fast(fabsf(r.dx) < eps ? copysignf(eps, r.dx) : r.dx);
    b.iy = rcp_fast(fabsf(r.dy) < eps ? copysignf(eps, r.dy) : r.dy);
    b.iz = rcp_fast(fabsf(r.dz) < eps ? copysignf(eps, r.dz) : r.dz);
    b.nx = -r.ox * b.ix;
    b.ny = -r.oy * b.iy;
    b.nz = -r.oz * b.iz;
    return b;
}

// Whether the ray meets a hierarchy box within [tmin, tlimit].  The planes'
// t are off by a few ulp of the origin's and the box's coordinates; the
// boxes are widened by more (bvh_build).
__device__ __forceinline__ bool box_hit(const BvhNode& B, const BoxRay& b, float tmin, float tlimit) {
    const float ax = fmaf(B.lo[0], b.ix, b.nx), bx = fmaf(B.hi[0], b.ix, b.nx);
    const float ay = fmaf(B.lo[1], b.iy, b.ny), by = fmaf(B.hi[1], b.iy, b.ny);
    const float az = fmaf(B.lo[2], b.iz, b.nz), bz = fmaf(B.hi[2], b.iz, b.nz);
    return fmaxf(max3f(fminf(ax, bx), fminf(ay, by), fminf(az, bz)), tmin) <=
           fminf(min3f(fmaxf(ax, bx), fmaxf(ay, by), fmaxf(az, bz)), tlimit);
}

// Nodes of the hierarchy with this root.
__device__ __forceinline__ uint32_t bvh_end(const BvhNode& root) { return (root.b & kBvhLeaf) ? 1u : root.a; }

// Whether the ray may enter frame F's root cell by tlimit, and then a t0 no
// later than it does: the root clip of frame_setup with the hardware
// reciprocal, each plane's t widened by more than the two can differ, so that
// no frame that a walk would enter is ruled out.  Plane by plane, because a
// direction along an axis has planes at 2^21 times the others' t, beside
// whose rounding every box on the ray's line would pass.
__device__ __forceinline__ bool may_enter(const FrameRec& F, const Ray& r, float tlimit, float& t0) {
    constexpr float kSlack = 0x1p-19f;
    FrameRay fr;
    frame_setup<false>(F, r, tlimit, fr, t0);
    const float N = (float)(1u << fr.K);
    auto exit_by = [&](float i, float b) {
        const float t = fmaf(N, i, b);
        return fmaf(fabsf(t) + fabsf(b), kSlack, t);
    };
    t0 = fmaf(-fabsf(t0), kSlack, t0);   // (grows with t0: the last plane entered stays the last)
    return t0 < INFINITY && t0 <= fminf(min3f(exit_by(fr.ix, fr.bx), exit_by(fr.iy, fr.by), exit_by(fr.iz, fr.bz)), tlimit);
}

__device__ __forceinline__ bool ray_valid(const Ray& r) {
    const bool fin = isfinite(r.ox) && isfinite(r.oy) && isfinite(r.oz) && isfinite(r.dx) && isfinite(r.dy) &&
                     isfinite(r.dz);
    const bool nonzero = max3f(fabsf(r.dx), fabsf(r.dy), fabsf(r.dz)) >= 0x1p-100f;
    return fin && nonzero && !isnan(r.tmin) && !isnan(r.tmax) && r.tmin <= r.tmax && r.tmin < INFINITY;
}

__host__ __device__ __forceinline__ size_t align16(size_t v) { return (v + 15) & ~(size_t)15; }

// Pointers read out of LDS job records lose their address space; these
// accessors restore it so the compiler emits global (not generic) loads and
// stores.
typedef float v4f __attribute__((ext_vector_type(4)));
typedef unsigned int v4u __attribute__((ext_vector_type(4)));

template <typename T>
__device__ __forceinline__ T gld(const T* p, uint64_t i) {
    return ((const __attribute__((address_space(1))) T*)p)[i];
}
// The 8-byte word at a 32-bit byte offset from a wave-uniform base (the
// scalar-base form of the load: no 64-bit address arithmetic per lane).
__device__ __forceinline__ uint64_t gld_at32(const uint64_t* p, uint32_t byte) {
    return *(const __attribute__((address_space(1))) uint64_t*)((const __attribute__((address_space(1))) char*)p + byte);
}
// Loads and stores with the streaming hint, for what this launch touches once.
// Hits always go out with it, so that they push fewer nodes out of the L2s:
// 1080p terrain under moving cameras 158 -> 150 us, instances 268 -> 260, their
// AO rays 428 -> 406 (a following pass over the hits is no slower).
template <typename T>
__device__ __forceinline__ T gld_once(const T* p, uint64_t i) {
    return __builtin_nontemporal_load((const __attribute__((address_space(1))) T*)p + i);
}
template <typename T>
__device__ __forceinline__ void gst_once(T* p, uint64_t i, T v) {
    __builtin_nontemporal_store(v, (__attribute__((address_space(1))) T*)p + i);
}
template <typename T>
__device__ __forceinline__ void gst(T* p, uint64_t i, T v) {
    ((__attribute__((address_space(1))) T*)p)[i] = v;
}

}  // namespace

// Per-lane candidate list in LDS: kCandList entries and the one after which
// the next list starts, an entry t and the candidate's place in the job's list
// (16 bits) each.  A constant length, as every address that depends on one
// read from the arguments costs a register in the kernel (1080p terrain 127.2
// and 131.9 us, a batch of 8 jobs 355 and 370).
constexpr uint32_t kCandEntryBytes = 64 * (4 + 2);   // of a wave
__host__ __device__ __forceinline__ uint32_t cand_bytes(const TraceArgs& a) {
    return a.max_cand ? (kCandList + 1u) * kCandEntryBytes : 0u;
}

// Traversal-stack slots per lane: slot sb + h holds the node whose children
// are the cells of size 2^h of the frame at base sb; the frame root's own
// level needs none.
__host__ __device__ __forceinline__ uint32_t stack_slots(const TraceArgs& a) { return a.stack_levels - 1u; }
__host__ __device__ __forceinline__ uint32_t stack_slot_bytes(const TraceArgs& a) { return a.wide ? 5u : 4u; }

size_t trace_lds_bytes(const TraceArgs& a, uint32_t waves_per_block) {
    const size_t shared = (size_t)a.n_frames * sizeof(FrameRec) + (size_t)a.n_cand_total * 16 +
                          align16((size_t)a.n_cand_total * 2) + (size_t)a.n_jobs * sizeof(JobRec) + (size_t)a.n_bvh_total * sizeof(BvhNode) + (a.jobs ? 0 : kHotLdsBytes) +
                          (a.has_cam0 ? sizeof(CameraArgs) : 0);
    const size_t per_wave = cand_bytes(a) + align16((size_t)stack_slots(a) * 64 * stack_slot_bytes(a)) +
                            (size_t)a.nest_levels * 64 * 16;
    return shared + per_wave * waves_per_block;
}

// kSorted: every job's candidates are tested one by one (at most 16 of
// them); otherwise through the per-frame box hierarchy.  A launch uses one of
// the two, and each instantiation carries only its own path.  All but one are
// compiled for 6 resident waves per SIMD (80 VGPRs): the few values that then
// go to scratch are per-ray state outside the walk loop, and the extra waves
// hide more of the node-load latency.  (12 waves a work-group, 2 work-groups a
// CU: hierarchy for 4 waves instances 309 us, their AO rays 490; for 5 waves
// 312 and 494; for 6 waves 260 and 394.  One-by-one for 7 waves: 1080p terrain
// 136 us, for 6 waves 126.)  The wide hierarchy one is compiled for 5 (96
// VGPRs): 4096^3 terrain, tuned, 1,507 us at 4 waves, 1,501 at 5, 1,611 at 6,
// where it spills more.
// kSingle: a one-job launch (the job in the arguments), whose pool and table
// offsets are then launch-wide values (scalar registers) rather than per-lane
// ones.
// kInline: the frame table comes in the arguments (TraceArgsInline).
// kWide: some pool of the launch has more than kPackedNodes nodes.  Its child
// starts do not fit the 24 bits beside a mask, so the stack keeps a 32-bit
// start and a mask byte apart (two LDS accesses and two addresses where the
// packed word takes one); smaller pools take the packed instantiations.
// kCount: the counting build (TraceArgs::counts and trail), for tests and
// measurement only.
template <bool kSorted, bool kSingle, bool kInline, bool kWide, bool kCount = false>
__global__ __launch_bounds__(1024) __attribute__((amdgpu_waves_per_eu(kSorted || !kWide ? 6 : 5, 8))) void trace_kernel(
    typename std::conditional<kInline, TraceArgsInline, TraceArgs>::type a) {
    extern __shared__ __align__(16) unsigned char smem[];
    unsigned char* p = smem;
    FrameRec* lds_frames = reinterpret_cast<FrameRec*>(p);
    p += (size_t)a.n_frames * 64;
    float4* lds_sph = reinterpret_cast<float4*>(p);
    p += (size_t)a.n_cand_total * 16;
    uint16_t* lds_cand = reinterpret_cast<uint16_t*>(p);
    p += align16((size_t)a.n_cand_total * 2);
    JobRec* lds_jobs = reinterpret_cast<JobRec*>(p);
    p += (size_t)a.n_jobs * sizeof(JobRec);
    BvhNode* lds_bvh = reinterpret_cast<BvhNode*>(p);
    p += (size_t)a.n_bvh_total * sizeof(BvhNode);
    // slow tiles first (single-job launches): the work-group's header and the
    // tiles it lists
    uint32_t* lds_hot = reinterpret_cast<uint32_t*>(p);
    if (kSingle) p += kHotLdsBytes;
    // a single job's camera (read once per claim; kept in LDS rather than in
    // scalar registers for the whole launch)
    CameraArgs* lds_cam = reinterpret_cast<CameraArgs*>(p);
    if (a.has_cam0) p += sizeof(CameraArgs);
    const uint32_t lane = threadIdx.x & 63u;
    const uint32_t wave = threadIdx.x >> 6;
    const size_t ent_bytes = cand_bytes(a);
    const size_t stack_bytes = (size_t)stack_slots(a) * 64 * (kWide ? 5 : 4);
    const size_t per_wave = ent_bytes + stack_bytes + (size_t)a.nest_levels * 64 * 16;
    unsigned char* wp = p + per_wave * wave;
    // traversal stack, slot l: the node word at stkc[l * 64]; kWide: the
    // child start there and the child mask at stkm[l * 64]
    uint32_t* stkc = reinterpret_cast<uint32_t*>(wp + ent_bytes) + lane;
    uint8_t* stkm = reinterpret_cast<uint8_t*>(wp + ent_bytes + (size_t)stack_slots(a) * 256) + lane;
    uint4* fst = reinterpret_cast<uint4*>(wp + ent_bytes + stack_bytes) + lane;  // nest n at fst[n * 64]

    // launch-wide counts: the arguments, or a plan's header (capacities
    // above bound them, so every LDS copy below stays in its region)
    uint64_t n_rays = a.n_rays;
    uint32_t n_jobs = a.n_jobs, n_frames = a.n_frames, n_cand_total = a.n_cand_total;
    uint32_t n_bvh = a.n_bvh_total;
    uint32_t tstride = (uint32_t)a.tile_stride;
    double tile_inv = a.tile_inv;
    if (a.hdr) {
        const LaunchHdr& h = *a.hdr;
        n_rays = h.n_rays;
        tstride = (uint32_t)h.tile_stride;
        tile_inv = h.tile_inv;
        n_jobs = min(h.n_jobs, a.n_jobs);
        n_frames = min(h.n_frames, a.n_frames);
        n_cand_total = min(h.n_cand_total, a.n_cand_total);
        n_bvh = min(h.n_bvh_total, a.n_bvh_total);
        if (n_jobs == 0) n_rays = 0;
    }
    // work-groups beyond what this launch's rays need (a plan's grid is
    // fixed) fill no LDS and claim nothing
    const uint32_t wpb = blockDim.x >> 6;
    const uint32_t n_tiles = (uint32_t)((n_rays + 63) >> 6);   // at most 0xff000000 / 64
    const uint32_t n_active = min(gridDim.x, (n_tiles + wpb - 1u) / wpb);
    const bool active = blockIdx.x < n_active;
    if (!active) {
        n_frames = 0;
        n_cand_total = 0;
        n_bvh = 0;
        n_jobs = 0;
    }
    // the frame table: in the arguments (small one-job launches) or in
    // device memory
    const FrameRec* src_frames = a.frames;
    const float4* src_sph = a.spheres;
    const uint32_t* src_cand = a.cand;
    const double* xmaps = a.xmaps;   // read only at hits: stays in global memory
    if constexpr (kInline) {
        src_frames = reinterpret_cast<const FrameRec*>(a.inline_tab);
        src_sph = reinterpret_cast<const float4*>(a.inline_tab + a.inline_off_sph);
        src_cand = reinterpret_cast<const uint32_t*>(a.inline_tab + a.inline_off_cand);
        xmaps = reinterpret_cast<const double*>(a.inline_tab + a.inline_off_x);
    }
    {
        const uint4* src = reinterpret_cast<const uint4*>(src_frames);
        uint4* dst = reinterpret_cast<uint4*>(lds_frames);
        for (uint32_t i = threadIdx.x; i < n_frames * 4u; i += blockDim.x) dst[i] = src[i];
    }
    for (uint32_t i = threadIdx.x; i < n_cand_total; i += blockDim.x) {
        lds_sph[i] = src_sph[i];
        lds_cand[i] = (uint16_t)src_cand[i];   // a launch holds at most 2047 frames
    }
    {
        const uint4* src = reinterpret_cast<const uint4*>(a.bvh);
        uint4* dst = reinterpret_cast<uint4*>(lds_bvh);
        for (uint32_t i = threadIdx.x; i < n_bvh * 2u; i += blockDim.x) dst[i] = src[i];
    }
    if (a.jobs) {
        const uint4* src = reinterpret_cast<const uint4*>(a.jobs);
        uint4* dst = reinterpret_cast<uint4*>(lds_jobs);
        for (uint32_t i = threadIdx.x; i < n_jobs * (uint32_t)(sizeof(JobRec) / 16); i += blockDim.x) dst[i] = src[i];
    } else if (threadIdx.x == 0) {
        lds_jobs[0] = a.job0;
    }
    if (kSingle && a.has_cam0 && threadIdx.x == 0) *lds_cam = a.cam0;
    // slow tiles first: the previous launch's list is this launch's input if
    // it traced the same rays (same signature); this launch's own slow tiles
    // go to the other list.  The state's header words stay fixed until the
    // last work-group out rewrites them, so each work-group reads them once
    // into its LDS header; the main loop reads the header there and the
    // state's pointer from the arguments, which keeps them out of its scalar
    // registers.
    if (kSingle && threadIdx.x < kHotLdsHdr) {
        const uint32_t* hot = a.hot;
        const uint32_t t = threadIdx.x;
        uint32_t v = 0;
        // (a launch with a tile or less per wave starts them all at once: no
        // order to choose, and its fixed claims need no queue)
        if (hot && !a.hdr && n_tiles <= kHotMaxTiles && n_tiles > n_active * wpb) {
            // one round of loads: the words of both lists, then the input's
            const uint32_t b = hot_in(hot);
            if (t == kHotLdsOn) {
                const bool same = ((uint64_t)hot[4 + 2 * b] | ((uint64_t)hot[5 + 2 * b] << 32)) == a.hot_sig;
                v = (!same || hot[10 + b] || a.hot_seq % kHotResample == 0) ? 1u : 0u;
            } else if (t == kHotLdsIn) {
                v = b;
            } else if (t == kHotLdsThr) {
                v = hot_thr(hot);
            } else if (t == kHotLdsDeal) {
                uint32_t c0 = 0, c1 = 0;
                for (uint32_t k = 0; k < kHotSub; ++k) {
                    c0 = max(c0, hot[kHotCntBase + k * kHotLine]);
                    c1 = max(c1, hot[kHotCntBase + (kHotSub + k) * kHotLine]);
                }
                const bool d0 = hot[10] && ((uint64_t)hot[4] | ((uint64_t)hot[5] << 32)) == a.hot_sig;
                const bool d1 = hot[11] && ((uint64_t)hot[6] | ((uint64_t)hot[7] << 32)) == a.hot_sig;
                // entry e is sub-list e mod kHotSub's (e / kHotSub)-th
                if (b ? d1 : d0) v = min(b ? c1 : c0, kHotSubCap) * kHotSub;
            } else if (t >= kHotLdsCnt && t < kHotLdsCnt + kHotSub) {
                const uint32_t k = t - kHotLdsCnt;
                const uint32_t c0 = hot[kHotCntBase + k * kHotLine], c1 = hot[kHotCntBase + (kHotSub + k) * kHotLine];
                v = min(b ? c1 : c0, kHotSubCap);
            } else if (t == kHotLdsPtr || t == kHotLdsPtr + 1) {
                v = (uint32_t)(reinterpret_cast<uint64_t>(hot) >> (t == kHotLdsPtr ? 0 : 32));
            }
        }
        lds_hot[t] = v;
    }
    __syncthreads();

    const uint32_t refill = a.refill;
    // partition q holds the claim slots s with s mod kQueueParts == q, so its
    // partition-local ray indices run to part_len(q) (whole tiles); a wave
    // owns the claimed range [rlo, rhi) of partition q (wave-uniform state).
    // Launches with fewer than two tiles per wave claim single tiles, so that
    // no wave waits for a second one while others have none.
    const uint32_t n_waves = n_active * wpb;
    const uint32_t claim = n_tiles < 2u * n_waves ? 64u : a.claim;
    auto part_len = [&](uint32_t p) -> uint32_t {
        return (n_tiles / kQueueParts + (p < n_tiles % kQueueParts ? 1u : 0u)) * 64u;
    };
    const uint32_t wave_id = blockIdx.x * wpb + wave;
    uint32_t q = wave_id % kQueueParts, rlo = 0, rhi = 0;
    // A launch of at most half the work-groups that its configuration lets
    // reside has a wave for every tile: wave w takes claim slot w, and the
    // queue is not used.  Such a launch is over in the time of a tile or two,
    // and a few atomic round trips (about 0.8 us each) to claim a tile and to
    // find the rest claimed are a good part of that (256x256 rays: 26.5 us
    // fixed, 29.7 by the counters; 100 rays 37.5 and 40.5).  A larger one
    // gains nothing by it (1080p: 157.5 either way), and where another
    // stream's launch still holds part of the device, its last work-groups
    // start late: tiles kept for them would wait.
    const bool fixed = 2u * n_active <= a.max_blocks;
    uint64_t known_dry = ~0ull;   // partitions this wave knows to be dry
    if (!fixed) {
        known_dry = __ballot(part_len(lane) == 0u);
    } else if (wave_id < n_tiles) {
        rlo = wave_id / kQueueParts * 64u;
        rhi = rlo + 64u;
    }
    // The tile that claim slot s covers: (s tstride) mod n_tiles, exactly (the
    // product stays below 2^53 and the quotient is off by at most one), in 15
    // instructions where the integer remainder takes about 80.
    auto tile_of = [&](uint32_t s) -> uint32_t {
        const double x = (double)s * (double)tstride;
        double rem = fma(-trunc(x * tile_inv), (double)n_tiles, x);
        if (rem < 0.0) rem += (double)n_tiles;
        if (rem >= (double)n_tiles) rem -= (double)n_tiles;
        return (uint32_t)rem;
    };

    // per-lane state
    uint32_t mode = M_DONE;
    uint32_t ri = 0;           // ray index within its job (a launch holds at most 0xff000000 rays)
    uint32_t gray = 0, c_nodes = 0, c_frames = 0, c_trail = 0;   // counting build only
    uint32_t job = 0;
    // a single job's constants come from its LDS copy, made wave-uniform:
    // read from the arguments, they would share one wide scalar load with
    // fields the loop never uses, and be kept or spilled with them
    const uint64_t* nodes = kSingle ? uniform_ptr(lds_jobs[0].nodes) : nullptr;
    uint32_t fbase = kSingle ? uniform_u32(lds_jobs[0].frame_base) : 0u;
    uint32_t cbase = kSingle ? uniform_u32(lds_jobs[0].cand_base) : 0u;
    uint32_t ncand = kSingle ? uniform_u32(lds_jobs[0].n_cand) : 0u;
    Ray r{};
    float best_t = INFINITY, tl = 0.f;
    uint32_t best_id = kNone, best_inst = kNone;
    int best_f = -1, best_axis = 3;
    uint32_t steps = 0;
    // the ray's candidate list: kUnlisted before it is made, then its length,
    // and kListMore if more candidates than it holds may have been tested
    uint32_t lst = kUnlisted;
    // entry k of the list is entered at lstt[k * 64] or later, its place in
    // the job's list is lstc[k * 64] (set where the list is used, so that the
    // walk keeps no registers for them)
    float* lstt = nullptr;
    uint16_t* lstc = nullptr;
    FrameRay fr{};
    // the current cell: corner (px, py, pz), size 2^h, reached at tc0; pw is
    // the word of its parent node (mask in the low byte, child start above;
    // kWide: the child start in pchild, the bits above the mask undefined)
    uint32_t cur_f = 0, pw = 0, pchild = 0, px = 0, py = 0, pz = 0, h = 0, nest = 0;
    // the current frame's stack slots start at fs (slot 0 of the frame: cells
    // of size 1).  The slot of size 2^h holds the node on the current path
    // whose children have that size: pw (and pchild) always copy the current
    // slot, so leaving cells up to any level is a plain read.  A frame
    // entered in place takes the slots below its cell's.
    uint32_t* fs = stkc;
    [[maybe_unused]] uint8_t* fsm = stkm;
    [[maybe_unused]] uint32_t cmask = ~0u;        // child start bits of a job's node words (kWide, several jobs)
    float tc0 = 0.f;
    // what the next walk step does first: PEND_RESUME continue just past a
    // transformed cell the walk came back from; PEND_ROOT_HIT the frame root
    // is itself a solid leaf (recorded where every walk hit is)
    uint32_t pend = 0;
    bool exhausted = !active;  // wave-uniform
    // slow tiles first: the tile the wave's lanes are tracing (whole-tile
    // refill; set only while the launch keeps the slow-tile state)
    uint32_t cur_tile = 0xFFFFFFFFu;

    auto record_hit = [&](float t, uint32_t id, uint32_t f, int axis) {
        const uint32_t inst = lds_frames[f].inst;
        if (t < best_t || (t == best_t && (inst < best_inst || (inst == best_inst && id < best_id)))) {
            best_t = t;
            best_id = id;
            best_inst = inst;
            best_f = (int)f;
            best_axis = axis;
            tl = fminf(r.tmax, best_t);
        }
    };

    // The children of node word w0 (child start c) become the cells walked,
    // of size 2^h: into the registers and their stack slot.
    auto set_node = [&](uint32_t w0, uint32_t c) {
        pw = w0;
        if constexpr (kWide) {
            pchild = c;
            fs[h * 64] = c;
            fsm[h * 64] = (uint8_t)w0;
        } else {
            fs[h * 64] = w0;
        }
    };
    // ... and back from their stack slot.
    auto load_node = [&]() {
        if constexpr (kWide) {
            pchild = fs[h * 64];
            pw = fsm[h * 64];
        } else {
            pw = fs[h * 64];
        }
    };
    // Stack slots from sb on; a frame record's root as a node word.
    auto set_slots = [&](uint32_t sb) {
        fs = stkc + sb * 64;
        if constexpr (kWide) fsm = stkm + sb * 64;
    };
    auto root_word = [&](const FrameRec& F) -> uint32_t { return kWide ? F.info : (F.child << 8) | (F.info & FR_MASK); };
    // First cell of a frame entered at t: the root's child that holds it.
    auto first_cell = [&](float t) {
        const float half = (float)(1u << h);
        px = (fmaf(half, fr.ix, fr.bx) <= t) ? (1u << h) : 0u;
        py = (fmaf(half, fr.iy, fr.by) <= t) ? (1u << h) : 0u;
        pz = (fmaf(half, fr.iz, fr.bz) <= t) ? (1u << h) : 0u;
        tc0 = t;
    };

    // Enter top-level frame f from its root.  Returns true when a walk starts.
    auto start_frame = [&](uint32_t f) -> bool {
        const FrameRec& F = lds_frames[f];
        if (F.info & FR_EMPTY) return false;
        float t0;
        if (!frame_setup<true>(F, r, tl, fr, t0)) return false;
        if constexpr (kCount) {
            ++c_frames;
            ++c_nodes;   // the frame's root record
        }
        cur_f = f;
        if (F.info & FR_ROOT_LEAF) {
            px = py = pz = 0u;
            h = fr.K;
            pend = PEND_ROOT_HIT;
            return true;
        }
        h = fr.K - 1u;
        set_slots(stack_slots(a) - fr.K);
        set_node(root_word(F), F.child);
        nest = 0;
        first_cell(t0);
        pend = 0;
        return true;
    };

    // Hit buffer (Sec. 4.3, for transforms on nodes): the outputs hold the
    // previous trace of this ray.  A previous hit in the static world frame
    // (or a miss) is still the answer unless some moved frame -- in place or
    // candidate -- now lies in front of it; the world frame itself never
    // changes.  Every moved frame (through the candidate hierarchy's boxes
    // when there is one) is tested up to the previous hit.
    auto previous_stands = [&]() -> bool {
        // a moved frame can hold a hit no later than tlim only if the ray
        // enters its root cell by then: the sphere first, then the root-cell
        // entry (leaf entries never precede it); c: place in the job's list
        auto may_reach = [&](uint32_t c, float tlim) -> bool {
            float t0;
            return sphere_may_hit(lds_sph[cbase + c], r, tlim) && may_enter(lds_frames[lds_cand[cbase + c]], r, tlim, t0);
        };
        const JobRec& J = lds_jobs[job];
        if (!J.out_inst) return false;
        const uint32_t pid = gld(J.out_id, ri);
        const uint32_t pinst = gld(J.out_inst, ri);
        const float pt = gld(J.out_t, ri);
        if (pinst != kNone || pid == kStepLimitId || isnan(pt)) return false;
        const float tlim = fminf(pt, r.tmax);
        const uint32_t nin = J.n_inline;
        for (uint32_t i = 0; i < nin; ++i)
            if (may_reach(ncand + i, tlim)) return false;
        if (ncand == 0) return true;
        if (kSorted) {
            for (uint32_t c = 0; c < ncand; ++c)
                if (may_reach(c, tlim)) return false;
            return true;
        }
        // any candidate box in front of the previous hit?
        const BoxRay br = box_ray(r);
        const BvhNode* bvh = lds_bvh + J.bvh_base;
        const uint32_t end = bvh_end(bvh[0]);
        for (uint32_t i = 0; i < end;) {
            const BvhNode& N = bvh[i];
            const bool leaf = (N.b & kBvhLeaf) != 0u;
            if (!box_hit(N, br, r.tmin, tlim)) {
                i = leaf ? i + 1u : N.a;
                continue;
            }
            if (leaf) {
                for (uint32_t c = N.a; c < N.a + (N.b & 0xFFFFu); ++c)
                    if (may_reach(c, tlim)) return false;
            }
            ++i;
        }
        return true;
    };

    // Test candidate c of the job for this ray and put it on its list of n:
    // of those tested, the nearest kCandList in order of entry and, where two
    // are entered at the same t, of their place.  more: of those that come
    // after entry kCandList.  By now the ray has its hit in the frames before,
    // if any, so candidates behind it drop out.
    auto list_candidate = [&](uint32_t c, bool more, uint32_t& n) {
        float t;
        if (!(sphere_may_hit(lds_sph[cbase + c], r, tl) && may_enter(lds_frames[lds_cand[cbase + c]], r, tl, t))) return;
        if (more) {
            const float from = lstt[kCandList * 64];
            if (t < from || (t == from && c <= lstc[kCandList * 64])) return;
        }
        uint32_t k = n;
        if (k == kCandList) {
            // in place of the last of them, if that comes after (equal ones
            // do not: candidates are tested in the order of their places)
            k = 0;
            for (uint32_t q = 1; q < kCandList; ++q) {
                const float v = lstt[q * 64], w = lstt[k * 64];
                if (v > w || (v == w && lstc[q * 64] > lstc[k * 64])) k = q;
            }
            if (!(t < lstt[k * 64])) return;
        }
        n = max(n, k + 1u);
        lstt[k * 64] = t;
        lstc[k * 64] = (uint16_t)c;
    };

    auto finish = [&]() {
        float nx = 0.f, ny = 0.f, nz = 0.f;
        if (best_id == kStepLimitId) {
            best_inst = kNone;
            best_t = INFINITY;
        } else if (best_f >= 0 && best_axis < 3) {
            // outward normal: -sgn(d_a) e_a in the frame, mapped by M^T (row a of M)
            const float* row = &lds_frames[best_f].m[4 * best_axis];
            const float da = fmaf(row[0], r.dx, fmaf(row[1], r.dy, row[2] * r.dz));
            const float s = (da < 0.f) ? 1.f : -1.f;
            const float inv = s * rsq_fast(fmaf(row[0], row[0], fmaf(row[1], row[1], row[2] * row[2])));
            nx = row[0] * inv;
            ny = row[1] * inv;
            nz = row[2] * inv;
        }
        const JobRec& J = lds_jobs[job];
        if constexpr (kCount) {
            gst(a.counts, (uint64_t)gray, c_nodes);
            gst(a.counts, n_rays + gray, c_frames);
            atomicAdd(a.counts + 2 * n_rays + gray, 1u);
        }
        gst_once(J.out_id, ri, best_id);
        if (J.out_inst) gst_once(J.out_inst, ri, best_inst);
        gst_once(J.out_t, ri, best_t);
        if (J.out_n) {
            gst_once(J.out_n, 3 * (uint64_t)ri, nx);
            gst_once(J.out_n, 3 * (uint64_t)ri + 1, ny);
            gst_once(J.out_n, 3 * (uint64_t)ri + 2, nz);
        }
        mode = M_DONE;
    };

    for (;;) {
        // ---------------------------------------------------------- refill
        const uint64_t idle = __ballot(mode == M_DONE);
        const uint32_t nidle = (uint32_t)__popcll(idle);
        if (nidle == 64u && cur_tile != 0xFFFFFFFFu) {
            // the wave's tile is done (whole tiles): listed when its slowest
            // ray took at least the threshold's advances
            const uint32_t m = wave_max(steps);
            steps = 0;   // lanes left without a ray in the next tile count nothing
            if (lane == 0u) {
                atomicAdd(lds_hot + kHotLdsSum, min(m, kHotCostClamp));
                atomicMax(lds_hot + kHotLdsMax, min(m, kHotCostClamp));
                if (m >= lds_hot[kHotLdsThr]) {
                    const uint32_t i = atomicAdd(lds_hot + kHotLdsListed, 1u);
                    if (i < kHotPerBlock) lds_hot[kHotLdsHdr + i] = cur_tile | (min(m, kHotEntryCostMax) << kHotTileBits);
                }
            }
            cur_tile = 0xFFFFFFFFu;
        }
        if (exhausted && nidle == 64u) break;
        if (!exhausted && nidle >= refill) {
            const uint32_t leader = (uint32_t)__ffsll((unsigned long long)idle) - 1u;
            bool retrace = false;
            // slow tiles first: whether this launch keeps the state, and
            // the input entries to deal out
            bool got_hot = false;
            uint32_t htile = 0, hcost = 0, hon = 0, hin = 0;
            if constexpr (kSingle) {
                hon = lds_hot[kHotLdsOn];
                hin = lds_hot[kHotLdsDeal];
            }
            if (hin && rlo >= rhi) {
                // the work-group's next entry, claimed by the leader for the
                // wave (hin and the counts stay fixed during the launch)
                const auto claim_entry = [&]() -> uint32_t {
                    uint32_t k = 0;
                    if (lane == leader) k = atomicAdd(lds_hot + kHotLdsTaken, 1u);
                    return (uint32_t)__builtin_amdgcn_readlane((int)k, (int)leader);
                };
                const uint32_t e = hot_deal(claim_entry, wpb, n_active, blockIdx.x, hin, lds_hot + kHotLdsCnt);
                if (e != kHotNone) {
                    got_hot = true;
                    const uint32_t sub = e % kHotSub, i = e / kHotSub;
                    const uint32_t ent = gld(hot_list(lds_hot_ptr(lds_hot), lds_hot[kHotLdsIn]), (uint64_t)sub * kHotSubCap + i);
                    htile = ent & kHotTileMask;
                    hcost = ent >> kHotTileBits;
                }
            }
            if constexpr (kSorted && kSingle) {
                // a dealt tile among the previous launch's costliest: its
                // wave issues ahead of the others on its SIMD while it runs
                // (a scalar branch: s_setprio ignores the lane mask)
                const bool up = got_hot && 10ull * hcost >= (uint64_t)kHotPrioTenths * lds_hot[kHotLdsThr];
                if (uniform_u32(up ? 1u : 0u)) __builtin_amdgcn_s_setprio(3);
                else __builtin_amdgcn_s_setprio(0);
            }
            if (!got_hot && rlo >= rhi) {
                // claim the next range of partition q.  The wave that takes a
                // partition's last range marks it in the shared bitmap, so a
                // set bit always means dry (an unset one may be stale); a wave
                // that finds its partition dry moves on to the next one it does
                // not know to be dry, and is done once it knows all of them
                // are.  (Reading the bitmap beside every claim, which saves a
                // round trip at the end, made the 1080p terrain 2 % slower.)
                uint32_t base = 0, len = 0;
                while (known_dry != ~0ull) {
                    uint64_t dry = 0;
                    len = part_len(q);
                    if (lane == leader) {
                        uint32_t* bm = a.queue + kQueueDry;
                        base = atomicAdd(a.queue + q * kQueueStride, claim);
                        if (base >= len)
                            dry = (uint64_t)__hip_atomic_load(bm, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) |
                                  ((uint64_t)__hip_atomic_load(bm + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) << 32);
                        else if (base + claim >= len)
                            atomicOr(bm + (q >> 5), 1u << (q & 31u));
                    }
                    base = __shfl(base, (int)leader);
                    if (base < len) break;
                    known_dry |= __shfl(dry, (int)leader) | (1ull << q);
                    if (known_dry == ~0ull) break;
                    // the next partition after q not known to be dry, cyclically
                    const uint64_t open = ~known_dry;
                    const uint64_t above = open & ~((2ull << q) - 1ull);
                    q = (uint32_t)__ffsll((unsigned long long)(above ? above : open)) - 1u;
                }
                if (known_dry == ~0ull) {
                    exhausted = true;
                } else {
                    rlo = base;
                    rhi = min(base + claim, len);
                }
            }
            const uint32_t take = got_hot ? min(nidle, 64u) : ((rlo < rhi) ? min(nidle, rhi - rlo) : 0u);
            const uint32_t first = rlo;
            if (!got_hot) rlo += take;
            // a regular claim's tile (whole tiles: the same for every lane)
            // and the input bitmap's word for it, tested once the rays'
            // loads are on their way
            const uint32_t csl = (first >> 6) * kQueueParts + q;
            const uint32_t ctile = tile_of(csl);
            uint32_t cword = 0;
            if (take && !got_hot && hin) cword = gld(hot_bits(lds_hot_ptr(lds_hot), lds_hot[kHotLdsIn]), ctile >> 5);
            if (mode == M_DONE) {
                const uint32_t rank =
                    __builtin_amdgcn_mbcnt_hi((uint32_t)(idle >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)idle, 0u));
                const uint32_t j = first + rank;
                const uint32_t slot = (j >> 6) * kQueueParts + q;     // claim order
                uint64_t gidx = n_rays;
                if (got_hot) {
                    if (rank < take && htile < n_tiles) gidx = (uint64_t)htile * 64u + rank;
                } else if (rank < take && slot < n_tiles) {
                    // a lane in the claim's first tile (every lane, with
                    // whole tiles) takes its tile from ctile
                    uint32_t tile = ctile;
                    if ((j >> 6) != (first >> 6)) tile = tile_of(slot);
                    gidx = (uint64_t)tile * 64u + (j & 63u);
                }
                if (gidx < n_rays) {
                    if constexpr (kCount) {
                        gray = (uint32_t)gidx;
                        c_nodes = c_frames = c_trail = 0;
                    }
                    const float4* rays;
                    const CameraArgs* cam = nullptr;
                    if constexpr (kSingle) {
                        ri = (uint32_t)(gidx - lds_jobs[0].ray_begin);
                        rays = lds_jobs[0].rays;
                    } else {
                        // the job holding this launch-wide ray index (jobs are in ray order)
                        uint32_t lo = 0, hi = n_jobs;
                        while (hi - lo > 1u) {
                            const uint32_t mid = (lo + hi) >> 1;
                            if (lds_jobs[mid].ray_begin <= gidx) lo = mid; else hi = mid;
                        }
                        job = lo;
                        const JobRec& J = lds_jobs[job];
                        ri = (uint32_t)(gidx - J.ray_begin);
                        nodes = J.nodes;
                        if constexpr (kWide) cmask = J.child_mask;
                        fbase = J.frame_base;
                        cbase = J.cand_base;
                        ncand = J.n_cand;
                        rays = J.rays;
                        cam = J.cam;
                    }
                    // the ray: read, or made from the job's camera (Fig. 5:
                    // one pixel sample per ray)
                    bool made = false;
                    if constexpr (kSingle) {
                        if (a.has_cam0) {
                            uint32_t w[sizeof(CameraArgs) / 4];
                            const uint32_t* src = reinterpret_cast<const uint32_t*>(lds_cam);
                            for (int k = 0; k < (int)(sizeof(CameraArgs) / 4); ++k) w[k] = uniform_u32(src[k]);
                            CameraArgs C;
                            std::memcpy(&C, w, sizeof C);
                            float4 c0, c1;
                            camera_ray(C, ri, c0, c1);
                            r = Ray{c0.x, c0.y, c0.z, c0.w, c1.x, c1.y, c1.z, c1.w};
                            made = true;
                        }
                    } else {
                        if (cam) {
                            // 96 bytes from global memory (six 16-byte loads)
                            v4u w[6];
                            for (int k = 0; k < 6; ++k) w[k] = gld(reinterpret_cast<const v4u*>(cam), k);
                            CameraArgs C;
                            std::memcpy(&C, w, sizeof C);
                            float4 c0, c1;
                            camera_ray(C, ri, c0, c1);
                            r = Ray{c0.x, c0.y, c0.z, c0.w, c1.x, c1.y, c1.z, c1.w};
                            made = true;
                        }
                    }
                    if (!made) {
                        const v4f* rp = reinterpret_cast<const v4f*>(rays);
                        v4f r0, r1;
                        if (kSingle && a.stream_rays) {
                            // between marks that keep the compiler from merging
                            // the two branches' loads, which would drop the hint
                            asm volatile("");
                            r0 = gld_once(rp, 2 * (uint64_t)ri);
                            r1 = gld_once(rp, 2 * (uint64_t)ri + 1);
                            asm volatile("");
                        } else {
                            r0 = gld(rp, 2 * (uint64_t)ri);
                            r1 = gld(rp, 2 * (uint64_t)ri + 1);
                        }
                        r = Ray{r0.x, r0.y, r0.z, r0.w, r1.x, r1.y, r1.z, r1.w};
                    }
                    best_t = INFINITY;
                    best_id = kNone;
                    best_inst = kNone;
                    best_f = -1;
                    best_axis = 3;
                    steps = 0;
                    lst = kUnlisted;
                    // a tile of the input list was traced by the wave it was dealt to
                    const bool dealt = !got_hot && ((cword >> (ctile & 31u)) & 1u);
                    bool keep = false;
                    if (!dealt && a.reuse && ray_valid(r)) keep = previous_stands();
                    if (dealt || keep) {
                        // nothing to trace or write: dealt to another wave, or
                        // the previous result stands
                    } else if (!ray_valid(r)) {
                        finish();
                    } else {
                        retrace = true;
                        tl = r.tmax;
                        mode = start_frame(fbase) ? M_WALK : M_SELECT;
                    }
                }
            }
            if (hon && take) {
                // wave-uniform
                const uint32_t t = got_hot ? (htile < n_tiles ? htile : 0xFFFFFFFFu)
                                           : ((csl < n_tiles && !((cword >> (ctile & 31u)) & 1u)) ? ctile : 0xFFFFFFFFu);
                cur_tile = (uint32_t)__builtin_amdgcn_readfirstlane((int)t);
            }
            if (a.reuse && a.retraced) {
                const uint64_t re = __ballot(retrace);
                if (lane == leader && re) atomicAdd(a.retraced, (unsigned long long)__popcll(re));
            }
        }

        // ---------------------------------------------------------- walk
        if (mode == M_WALK) {
            // The octant of the current cell in its parent (bit h of each
            // corner, unmirrored), and whether the parent has that child.
            uint32_t oct = 0;
            auto occupied = [&]() -> uint32_t {
                oct = (__builtin_amdgcn_ubfe(px, h, 1) | (__builtin_amdgcn_ubfe(py, h, 1) << 1) |
                       (__builtin_amdgcn_ubfe(pz, h, 1) << 2)) ^ fr.flip;
                return __builtin_amdgcn_ubfe(pw, oct, 1);
            };
            uint32_t ev = EV_NONE;
            uint32_t evd = 0;   // the leaf hit, or the frame to enter
            const bool hit_root = pend == PEND_ROOT_HIT;
            // PEND_RESUME: continue just past a transformed cell the walk
            // came back from, as past an empty one
            uint32_t full = occupied();
            if (pend != 0u) full = 0u;
            pend = 0;
            if (hit_root) {
                ev = EV_HIT;
                evd = lds_frames[cur_f].root;
            }
            // The hot loop, until something happens.  Bound by VALU issue
            // while tiles are left and by the chain of one lane's turns at the
            // end.  Each turn leaves the current cell if it is empty, then
            // descends into the cell it now stands in if that one is not: some
            // lane of a wave needs either half on most turns, so a lane that
            // needs one after the other gets both from one turn.  Per 64-ray
            // tile of the 1080p terrain that is 14.4 turns running the halves
            // 12.1 and 12.9 times; a loop of one step (advance or descend) per
            // turn took 19.5 turns and 15.0 and 15.8 halves, and a second
            // advance per turn runs more instructions than it saves.  A turn
            // that runs both halves is 87 VALU instructions (about 115 with
            // child offsets relative to the node, the child start and mask
            // apart in the stack and the exit planes computed for both
            // halves).  Measured
            // against that loop: 1080p terrain animation 176 -> 145 us,
            // 4096^3 terrain at 4K 2,186 -> 1,846 us, 1080p instances 401 ->
            // 334 us, 256x256 sphere 64 -> 54 us.
            //
            // Everything that decides a lane's course (full, ev) is a number in
            // a vector register, and the advance half has no branch of its own:
            // a lane that stops there computes a state that nothing reads.  As
            // lane masks and branches the same loop took 67 scalar
            // instructions per turn, which a lone wave waits for one by one;
            // now it takes 34.  1080p terrain animation 144 -> 136 us, moving
            // camera 181 -> 167 us, 100 rays 44 -> 40 us.
            while (ev == EV_NONE) {
                if (full == 0u) {
                    // advance: leave the cell through its nearest exit
                    // plane(s); the new cell's size is 2^h2, h2 the highest
                    // changed corner bit (no plane at tc1, a NaN, changes
                    // none and ends the walk).  Descents between two advances
                    // are bounded by the depth, so counting advances bounds
                    // the walk.
                    const uint32_t size = 1u << h;
                    const uint32_t qx = px + size, qy = py + size, qz = pz + size;
                    const float ex = fmaf((float)qx, fr.ix, fr.bx);
                    const float ey = fmaf((float)qy, fr.iy, fr.by);
                    const float ez = fmaf((float)qz, fr.iz, fr.bz);
                    const float tc1 = min3f(ex, ey, ez);
                    const uint32_t nx = (ex == tc1) ? qx : px;
                    const uint32_t ny = (ey == tc1) ? qy : py;
                    const uint32_t nz = (ez == tc1) ? qz : pz;
                    const uint32_t diff = (nx ^ px) | (ny ^ py) | (nz ^ pz);
                    uint32_t lz = diff ? (uint32_t)__builtin_clz(diff) : ~0u;
                    opaque(lz);   // (one v_ffbh; folded into the line below it is three instructions)
                    const uint32_t h2 = 31u - lz;
                    ++steps;
                    // past the frame or the best hit, or out of steps: the
                    // lane stops (its state below is dead but for h and tc0,
                    // which tell the two apart; its stack read stays in range)
                    const bool on = tc1 <= tl && h2 < fr.K && steps <= a.step_limit;
                    const uint32_t keep = ~0u << (h2 & 31u);
                    px = nx & keep;
                    py = ny & keep;
                    pz = nz & keep;
                    h = min(h2, fr.K - 1u);
                    tc0 = tc1;
                    load_node();
                    full = occupied();
                    h = h2;
                    if (!on) full = 0u;
                    ev = on ? EV_NONE : EV_END;
                }
                opaque(full);
                if (full != 0u) {
                    // descend: the child's node word.  (A copy of the pool's
                    // first nodes in LDS took seven more instructions per
                    // turn to choose between the two and to fill, and the
                    // vector cache holds those nodes as well: 160.7 us with it
                    // and 157.5 us without on the 1080p terrain under a moving
                    // camera, instances 298 and 282 us, 100 rays 38.7 and 37.2.)
                    evd = (kWide ? pchild : pw >> 8) + __popc(__builtin_amdgcn_ubfe(pw, 0, oct));
                    const uint64_t w = kWide ? gld(nodes, evd) : gld_at32(nodes, evd * 8u);
                    if constexpr (kCount) {
                        if (a.trail && c_trail < a.trail_cap)
                            gst(a.trail, (uint64_t)c_trail * n_rays + gray, evd);
                        ++c_trail;
                        ++c_nodes;
                    }
                    const uint32_t w0 = (uint32_t)w;
                    const uint32_t w1 = (uint32_t)(w >> 32);
                    if (w0 - 1u < kNodeXform - 1u) {
                        // an interior node: into the child that holds the
                        // ray's point at tc0
                        h -= 1u;
                        const uint32_t hs = 1u << h;
                        const uint32_t cx = px | hs, cy = py | hs, cz = pz | hs;
                        px = (fmaf((float)cx, fr.ix, fr.bx) <= tc0) ? cx : px;
                        py = (fmaf((float)cy, fr.iy, fr.by) <= tc0) ? cy : py;
                        pz = (fmaf((float)cz, fr.iz, fr.bz) <= tc0) ? cz : pz;
                        set_node(w0, (kSingle || !kWide) ? w1 : (w1 & cmask));
                        full = occupied();
                    } else {
                        // a leaf, or a transformed node: a frame entered in
                        // place, or a candidate (traced on its own, empty here)
                        full = 0u;
                        ev = EV_HIT;
                        if (w0 != 0u) {
                            evd = fbase + 1u + w1;
                            ev = (lds_frames[evd].info & FR_INLINE) ? EV_ENTER : EV_NONE;
                        }
                    }
                }
                opaque(ev);
                opaque(full);
            }
            opaque(ev);   // the tests below are not the loop's
            if (ev == EV_END && tc0 <= tl && h < fr.K) ev = EV_LIMIT;
            if (ev == EV_HIT) {
                // the first solid leaf front to back ends this top-level frame;
                // a leaf the ray passes by in FP64 is empty for this ray (the
                // walk goes on past it; a frame root leaf ends the frame)
                int ha;
                float th;
                if (exact_hit(xmaps + (size_t)kExactMapDoubles * cur_f, r, fr, px, py, pz, 1u << h, th, ha)) {
                    record_hit(th, evd, cur_f, ha);
                    mode = M_SELECT;
                    nest = 0;
                } else if (hit_root) {
                    mode = M_SELECT;
                    nest = 0;
                } else {
                    pend = PEND_RESUME;
                }
            } else if (ev == EV_LIMIT) {
                best_id = kStepLimitId;
                finish();
            } else if (ev == EV_ENTER) {
                const FrameRec& C = lds_frames[evd];
                FrameRay cfr;
                float t0;
                // no later than the ray's way out of the cell
                const float cell_out = min3f(fmaf((float)(px + (1u << h)), fr.ix, fr.bx), fmaf((float)(py + (1u << h)), fr.iy, fr.by),
                                             fmaf((float)(pz + (1u << h)), fr.iz, fr.bz));
                if (frame_setup<true>(C, r, fminf(tl, cell_out), cfr, t0)) {
                    if constexpr (kCount) {
                        ++c_frames;
                        ++c_nodes;   // the frame's root record
                    }
                    // save where the enclosing walk stands (its current slot
                    // keeps its node), then enter in place
                    const uint32_t sb = (uint32_t)(fs - stkc) >> 6;
                    fst[nest * 64] = make_uint4(cur_f | (h << 11) | (sb << 16), px, py, pz);
                    ++nest;
                    cur_f = evd;
                    fr = cfr;
                    set_slots(sb + h - fr.K);
                    h = fr.K - 1u;
                    set_node(root_word(C), C.child);
                    first_cell(t0);
                } else {
                    pend = PEND_RESUME;  // missed it: the cell is empty for this ray
                }
            } else if (ev == EV_END) {
                if (nest > 0) {
                    // back to the enclosing frame, just past the transformed cell
                    --nest;
                    const uint4 e = fst[nest * 64];
                    cur_f = e.x & 0x7FFu;
                    h = (e.x >> 11) & 31u;
                    set_slots((e.x >> 16) & 127u);
                    px = e.y;
                    py = e.z;
                    pz = e.w;
                    float t0;
                    frame_setup<true>(lds_frames[cur_f], r, tl, fr, t0);
                    load_node();
                    pend = PEND_RESUME;
                } else {
                    mode = M_SELECT;
                }
            }
        }
        if (mode == M_SELECT) {
            // the walk's state is dead here (start_frame sets all of it before
            // the next walk step); saying so frees its registers for the
            // candidate search
            fr = FrameRay{};
            px = py = pz = h = 0;
            pw = pchild = 0;
            fs = stkc;
            fsm = stkm;
            cur_f = nest = 0;
            tc0 = 0.f;
            pend = 0;
            if (++steps > a.step_limit) {
                best_id = kStepLimitId;
                finish();
                continue;
            }
            // ------------------------------------------------------ next candidate frame
            // List the candidates the ray may enter before its best hit, the
            // nearest first (the first time here, and again past a full list):
            // each by its bounding sphere (Sec. 4.1) and its root-cell entry.
            // Listing after the walk of the static world instead of when the
            // ray was claimed lets that hit rule most of them out, and the
            // list stays short (1080p terrain: 0.08 entries per ray for 8
            // candidates).
            uint32_t l = lane;
            opaque(l);
            lstt = reinterpret_cast<float*>(wp) + l;
            lstc = reinterpret_cast<uint16_t*>(wp + (kCandList + 1u) * 256u) + l;
            uint32_t n = lst & 0xFFu;
            if (lst == kUnlisted || (n == 0u && lst != 0u)) {
                const bool more = lst != kUnlisted;
                n = 0;
                if constexpr (kSorted) {
                    for (uint32_t c = 0; c < ncand; ++c) list_candidate(c, more, n);
                } else if (ncand) {
                    // The job's box hierarchy in preorder, each lane for
                    // itself: a box that its ray misses is skipped with its
                    // subtree, which needs no stack.  One node at a time for
                    // the whole wave costs as much where its rays keep
                    // together (1080p instances 262 us either way, their AO
                    // rays 395), but visits the union of their boxes where
                    // they do not: 100 rays from anywhere against 1,000
                    // candidates 399 us, this walk 197; 400,000 against 250
                    // 352 and 243.
                    const BoxRay br = box_ray(r);
                    const BvhNode* bvh = lds_bvh + (kSingle ? uniform_u32(lds_jobs[0].bvh_base) : lds_jobs[job].bvh_base);
                    const uint32_t end = bvh_end(bvh[0]);
                    for (uint32_t i = 0; i < end;) {
                        const BvhNode& N = bvh[i];
                        const uint32_t na = N.a, nb = N.b;
                        const bool hit = box_hit(N, br, r.tmin, tl), leaf = (nb & kBvhLeaf) != 0u;
                        if (hit && leaf)
                            for (uint32_t c = na; c < na + (nb & 0xFFFFu); ++c) list_candidate(c, more, n);
                        i = (hit || leaf) ? i + 1u : na;
                    }
                }
                lst = (n == kCandList && n < ncand) ? kListMore : 0u;
            }
            float near = INFINITY;
            uint32_t at = 0;
            for (uint32_t k = 0; k < n; ++k) {
                const float v = lstt[k * 64];
                if (v < near || (v == near && lstc[k * 64] < lstc[at * 64])) {
                    near = v;
                    at = k;
                }
            }
            if (n == 0u || near > tl) {
                // none left, or the nearest lies beyond the best hit, and so
                // do the others
                finish();
            } else {
                const uint32_t c = lstc[at * 64];
                --n;
                lstt[at * 64] = lstt[n * 64];
                lstc[at * 64] = lstc[n * 64];
                lst = (lst & kListMore) | n;
                if (lst == kListMore) {
                    // the next list starts after this one
                    lstt[kCandList * 64] = near;
                    lstc[kCandList * 64] = (uint16_t)c;
                }
                if (start_frame(lds_cand[cbase + c])) {
                    mode = M_WALK;
                } else {
                    // a frame that the walk's own entry test misses, which is
                    // narrower than the list's, is no selection
                    --steps;
                }
            }
        }
    }

    // the last work-group out resets the queue for the next launch; only
    // work-groups that may claim count (an idle one of a plan's fixed grid
    // touches no counter, and skipping its atomic spares the others a
    // same-address queue), and none in a launch that used no counter.  Every
    // word that another work-group reads here is written by atomics, so all
    // that has to come before the count is their completion: each wave waits
    // for its own, and no cache is written back or invalidated (a device
    // fence here did both once per work-group: 140.0 against 137.3 us per
    // 1080p terrain frame).
    wait_memory();
    __syncthreads();
    uint32_t* const hot = (kSingle && lds_hot[kHotLdsOn]) ? a.hot : nullptr;
    const uint32_t hp = hot ? lds_hot[kHotLdsIn] : 0u, ob = hp ^ 1u;
    if (hot && active && threadIdx.x == 0) {
        // this work-group's slow tiles into the output list and its bitmap
        const uint32_t sub = blockIdx.x % kHotSub;
        atomicAdd(hot_sum(hot, sub), lds_hot[kHotLdsSum]);
        atomicMax(hot_max(hot, sub), lds_hot[kHotLdsMax]);
        const uint32_t n = min(lds_hot[kHotLdsListed], kHotPerBlock);
        if (n) {
            const uint32_t base = atomicAdd(hot_cnt(hot, ob, sub), n);
            uint32_t* olist = hot_list(hot, ob) + sub * kHotSubCap;
            uint32_t* obits = hot_bits(hot, ob);
            for (uint32_t i = 0; i < n && base + i < kHotSubCap; ++i) {
                const uint32_t ent = lds_hot[kHotLdsHdr + i], t = ent & kHotTileMask;
                olist[base + i] = ent;
                atomicOr(obits + (t >> 5), 1u << (t & 31u));
            }
        }
    }
    if (active && !fixed && threadIdx.x == 0) {
        wait_memory();
        uint32_t* fin = a.queue + kQueueFinished;
        const uint32_t prev = atomicAdd(fin, 1u);
        const bool last = prev == n_active - 1;
        if (last) {
            for (uint32_t p = 0; p < kQueueParts; ++p) atomicExch(a.queue + p * kQueueStride, 0u);
            atomicExch(a.queue + kQueueDry, 0u);
            atomicExch(a.queue + kQueueDry + 1, 0u);
            atomicExch(fin, 0u);
        }
        if (hot) lds_hot[kHotLdsListed] = last ? 1u : 0u;
    }
    if (hot) {
        __syncthreads();
        if (active && lds_hot[kHotLdsListed]) {
            // last out (every other work-group has written its list): clear
            // the input list's bitmap, the words of the tiles of the launch
            // that wrote it
            const uint32_t iw = (min(hot[12 + hp], kHotMaxTiles) + 31u) >> 5;
            uint32_t* ibits = hot_bits(hot, hp);
            for (uint32_t i = threadIdx.x; i < iw; i += blockDim.x) ibits[i] = 0u;
            if (threadIdx.x < 64u) {
                // the lines' counts and cost statistics, one line per lane
                const uint32_t k = threadIdx.x;
                uint32_t c = 0, csum = 0, cmax = 0;
                if (k < kHotSub) {
                    c = atomicAdd(hot_cnt(hot, ob, k), 0u);
                    csum = atomicExch(hot_sum(hot, k), 0u);
                    cmax = atomicExch(hot_max(hot, k), 0u);
                    atomicExch(hot_cnt(hot, hp, k), 0u);
                }
                for (int off = kHotSub / 2; off > 0; off >>= 1) {
                    c += (uint32_t)__shfl_xor((int)c, off);
                    csum += (uint32_t)__shfl_xor((int)csum, off);
                    cmax = max(cmax, (uint32_t)__shfl_xor((int)cmax, off));
                }
                if (k == 0u) {
                    // the threshold follows the target count of listed tiles
                    const uint32_t tg = a.hot_target, hthr = lds_hot[kHotLdsThr];
                    uint32_t nt = hthr;
                    if (c > tg + tg / 2u) nt = hthr + max(1u, hthr / 8u);
                    else if (2u * c < tg && hthr > 1u) nt = hthr - max(1u, hthr / 8u);
                    atomicExch(hot + 4 + 2 * ob, (uint32_t)a.hot_sig);
                    atomicExch(hot + 5 + 2 * ob, (uint32_t)(a.hot_sig >> 32));
                    // deal the new list out only if this launch was bound by
                    // its slowest tiles: largest cost >= 0.7 x (sum of costs /
                    // waves)
                    atomicExch(hot + 10 + ob, (10ull * cmax * n_active * wpb >= 7ull * csum) ? 1u : 0u);
                    atomicExch(hot + 12 + ob, (uint32_t)n_tiles);
                    atomicExch(hot + 1, nt);
                    atomicExch(hot + 0, ob);
                }
            }
        }
    }
}

// The allocation-free entry point's scratch (see static_scratch).  In host
// code this name is not a device address: host code reaches the array only
// through the pointer static_scratch returns.
__device__ __align__(256) unsigned char scratch[kStaticScratchBytes];

hipError_t static_scratch(int device, unsigned char** out) {
    constexpr int kMaxDevices = 64;
    static std::mutex mu;
    static unsigned char* addr[kMaxDevices] = {};
    if (device < 0 || device >= kMaxDevices || !out) return hipErrorInvalidValue;
    std::lock_guard<std::mutex> lock(mu);
    if (!addr[device]) {
        void* p = nullptr;
        const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess) return e;
        if (!p) return hipErrorInvalidSymbol;
        addr[device] = static_cast<unsigned char*>(p);
    }
    *out = addr[device];
    return hipSuccess;
}

__global__ __launch_bounds__(256) void zero_words_kernel(uint32_t* p, uint32_t n) {
    for (uint32_t i = blockIdx.x * blockDim.x + threadIdx.x; i < n; i += gridDim.x * blockDim.x) p[i] = 0u;
}

hipError_t launch_zero_words(uint32_t* p, uint32_t n, hipStream_t stream) {
    if (n == 0) return hipSuccess;
    hipLaunchKernelGGL(zero_words_kernel, dim3((n + 255) / 256 < 64 ? (n + 255) / 256 : 64), dim3(256), 0, stream, p, n);
    return hipGetLastError();
}

namespace {

// The instantiation of a launch, to be launched or to have its attributes
// set (f takes the kernel and whether it takes a TraceArgsInline).
template <bool kWide, typename F>
hipError_t with_kernel(bool sorted, bool single, bool inline_tab, bool count, F&& f) {
    if (count) {
        if (inline_tab) return f(&trace_kernel<true, true, true, kWide, true>);
        return sorted ? f(&trace_kernel<true, true, false, kWide, true>) : f(&trace_kernel<false, true, false, kWide, true>);
    }
    if (inline_tab) return f(&trace_kernel<true, true, true, kWide>);
    if (sorted) return single ? f(&trace_kernel<true, true, false, kWide>) : f(&trace_kernel<true, false, false, kWide>);
    return single ? f(&trace_kernel<false, true, false, kWide>) : f(&trace_kernel<false, false, false, kWide>);
}

template <typename F>
hipError_t with_kernel(bool wide, bool sorted, bool single, bool inline_tab, bool count, F&& f) {
    return wide ? with_kernel<true>(sorted, single, inline_tab, count, f)
                : with_kernel<false>(sorted, single, inline_tab, count, f);
}

}  // namespace

hipError_t prepare_trace(size_t max_lds) {
    const auto set = [&](auto* k) {
        return hipFuncSetAttribute(reinterpret_cast<const void*>(k), hipFuncAttributeMaxDynamicSharedMemorySize, (int)max_lds);
    };
    for (int v = 0; v < 32; ++v) {
        const hipError_t e = with_kernel((v & 1) != 0, (v & 2) != 0, (v & 4) != 0, (v & 8) != 0, (v & 16) != 0, set);
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

hipError_t launch_trace(const TraceArgs& a, const LaunchCfg& c, hipStream_t stream, const unsigned char* inline_tab,
                        size_t inline_bytes) {
    const dim3 grid(c.blocks), block(c.waves_per_block * 64);
    const bool count = a.counts != nullptr;
    if (count && (a.jobs || a.hdr)) return hipErrorInvalidValue;
    if (inline_tab && (!a.sort_cand || a.jobs || inline_bytes > kInlineTableBytes)) return hipErrorInvalidValue;
    return with_kernel(a.wide != 0, a.sort_cand != 0, !a.jobs, inline_tab != nullptr, count, [&](auto* k) {
        if constexpr (std::is_invocable_v<decltype(k), TraceArgsInline> && !std::is_invocable_v<decltype(k), TraceArgs>) {
            TraceArgsInline ai{};
            static_cast<TraceArgs&>(ai) = a;
            std::memcpy(ai.inline_tab, inline_tab, inline_bytes);
            hipLaunchKernelGGL(k, grid, block, c.lds_bytes, stream, ai);
        } else {
            hipLaunchKernelGGL(k, grid, block, c.lds_bytes, stream, a);
        }
        return hipGetLastError();
    });
}

}  // namespace svo
