// Full validation of listed edges (Alg. 1, the branch taken when not lazy:
// every edge left unknown gets a full collision check).
//
// The check is continuous: does any configuration q(t), t in [0, 1], of the
// edge's motion put a robot sphere into a present box?  It refines the two
// approximations of Sec. 3.2 on dyadic sub-intervals [j 2^-l, (j+1) 2^-l]:
//   free(l, j)  every sphere's capsule from its centre at the interval's start
//               to its centre at the end, radius r_i + delta_i 4^-l, misses
//               every present box (delta_i 4^-l bounds the chord deviation
//               over an interval of length 2^-l, since delta_i bounds
//               max|p''|/8 over the edge);
//   hit(t)      some sphere at q(t) meets a present box.
// Level by level: hit(0) or hit(1) -> COLLIDES (witness 0, then 1); free(0, 0)
// -> FREE at level 0; then with A_0 = {0} and l = 0, 1, ...: more than
// max_active unknown intervals -> UNRESOLVED at l; a midpoint of A_l hits ->
// COLLIDES at l+1, witness the smallest such midpoint; A_{l+1} = the children
// that are not free; none -> FREE at l+1; after max_level levels ->
// UNRESOLVED.
//
// The configurations use the build's binary64 motion parameters and a sin/cos
// made of a fixed sequence of binary64 +, -, * and rint (Cody and Waite's
// reduction by pi/2, Taylor series to degree 19/20), compiled without
// contraction, so any IEEE evaluator of the same steps reaches the same
// verdicts.  The distance predicates are the binary64 definitions of the
// update kernels (predicates64.h).
//
// One wavefront validates one listed edge at a time (grid-stride over the
// list).  Its present boxes near the edge are staged in LDS: a box
// can matter only if it meets the box around the edge's chords widened by
// r_i + 2 delta_i (each sub-chord stays within delta_i of the edge's chord,
// each sub-capsule adds at most r_i + delta_i), plus a rounding margin.  More
// than 64 such boxes are handled in pages.
#include <hip/hip_runtime.h>
#include <math.h>

#include "predicates64.h"
#include "rgg_device.h"

namespace rgg {

namespace {

constexpr int kVWaves = 4;         // wavefronts per block, an edge each
constexpr int kVT = 64 * kVWaves;  // threads per block
static_assert(kValBoxes == 64, "a lane marks a page's boxes in 64 bits, and stages one of them");
constexpr int kNoHit = 0x7fffffff;

__device__ inline void wave_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

constexpr uint8_t kFree = RGG_VERDICT_FREE;
constexpr uint8_t kCollides = RGG_VERDICT_COLLIDES;
constexpr uint8_t kUnresolved = RGG_VERDICT_UNRESOLVED;

// ---- configurations --------------------------------------------------------

// sin and cos: x = k (pi/2) + r with pi/2 split into a 24-bit head (exact
// products with k) and its binary64 remainder; Taylor series of sin r to r^19
// and cos r to r^20 in Horner form; the quadrant k mod 4 maps the pair.
__device__ inline void vsincos(double x, double *sn, double *cs)
{
    const double pi = 3.14159265358979323846;
    const double half_pi = pi / 2.0;
    const double head = (double)(float)half_pi;
    const double tail = half_pi - head;
    const double k = rint(x * (2.0 / pi));
    const double r = (x - k * head) - k * tail;
    const double z = r * r;
    double ps = -1.0 / 121645100408832000.0;
    ps = ps * z + 1.0 / 355687428096000.0;
    ps = ps * z - 1.0 / 1307674368000.0;
    ps = ps * z + 1.0 / 6227020800.0;
    ps = ps * z - 1.0 / 39916800.0;
    ps = ps * z + 1.0 / 362880.0;
    ps = ps * z - 1.0 / 5040.0;
    ps = ps * z + 1.0 / 120.0;
    ps = ps * z - 1.0 / 6.0;
    const double s = r + (r * z) * ps;
    double pc = 1.0 / 2432902008176640000.0;
    pc = pc * z - 1.0 / 6402373705728000.0;
    pc = pc * z + 1.0 / 20922789888000.0;
    pc = pc * z - 1.0 / 87178291200.0;
    pc = pc * z + 1.0 / 479001600.0;
    pc = pc * z - 1.0 / 3628800.0;
    pc = pc * z + 1.0 / 40320.0;
    pc = pc * z - 1.0 / 720.0;
    pc = pc * z + 1.0 / 24.0;
    pc = pc * z - 1.0 / 2.0;
    const double c = 1.0 + z * pc;
    const int64_t quadrant = (int64_t)k & 3;
    if (quadrant == 0) {
        *sn = s;
        *cs = c;
    } else if (quadrant == 1) {
        *sn = c;
        *cs = -s;
    } else if (quadrant == 2) {
        *sn = -s;
        *cs = -c;
    } else {
        *sn = -c;
        *cs = s;
    }
}

// ---- the kernel ------------------------------------------------------------

// LDS of one block, laid out by the host for the robot and the limits of the
// call: a planar robot of few spheres then leaves room for more edges in
// flight.  The robot and the resident boxes come first, then one region per
// wavefront (offsets within the region: doubles, then 32-bit words).
struct ValLds {
    int pos, rad, len, link, tile;                // block: robot (doubles; link: words), boxes
    int region0, region;                          // first region, doubles per region
    int mot, del, box, box32, list, cen, fk;      // doubles (list: 16-bit slots)
    int act, nxt;                                 // 32-bit words
    int bytes;
    int chunk;       // intervals refined together
    int fkw;         // doubles per configuration at fk
};

constexpr int kVChunkMax = 8;        // intervals per chunk at most (16 child flags in one word)
constexpr int kVCenDoubles = 400;    // sphere centres of a chunk (more when one interval needs it)
constexpr int kVTile = 512;          // resident boxes kept in LDS; more are scanned in memory
constexpr int kVCull = 16;        // candidates from which a step looks for ones to drop
constexpr int kVList = 256;          // candidate slots listed; more are found again page by page
static_assert(kVList % kValBoxes == 0 && kMaxSlots <= 65536, "whole pages are listed, as 16-bit slots");

constexpr ValLds val_lds(const ValDev &v, int max_active)
{
    ValLds l = {};
    const int sincos = v.kind == RGG_PLANAR_ARM ? v.L : (v.kind == RGG_SE3 ? 2 : 1);
    l.fkw = v.kind == RGG_PLANAR_ARM ? 4 * v.L : 2;
    // as many intervals as keep one lane per sine-cosine pair of their three
    // configurations, within the room for their centres
    int c = 64 / (3 * sincos);
    if (c > kVChunkMax) c = kVChunkMax;
    if (c > kVCenDoubles / (3 * v.B * v.D)) c = kVCenDoubles / (3 * v.B * v.D);
    l.chunk = c < 1 ? 1 : c;
    int d = 0;
    auto take = [&](int n) {
        const int at = d;
        d += n + (n & 1);                         // 16-byte steps
        return at;
    };
    l.pos = take(v.B * (v.kind == RGG_SE2 ? 2 : (v.kind == RGG_SE3 ? 3 : 1)));
    l.rad = take(v.B);
    l.len = take(v.L);
    l.link = 2 * take((v.B + 1) / 2);
    l.tile = take(v.M <= kVTile ? (int)v.M * v.D : 0);   // 2 D floats a box
    l.region0 = d;
    d = 0;
    const int page = (int)(v.M < kValBoxes ? (v.M > 0 ? v.M : 1) : kValBoxes);
    l.cen = take(3 * l.chunk * v.B * v.D);
    l.fk = take(3 * l.chunk * l.fkw);
    l.box32 = take(page * v.D);
    l.box = take(page * 2 * v.D);
    l.list = take((int)(v.M < kVList ? v.M : kVList) / 4 + 1);
    l.mot = take(v.vstride);
    l.del = take(v.B);
    l.act = 2 * d;
    l.nxt = l.act + max_active;
    d += max_active;
    d += d & 1;
    l.region = d;
    l.bytes = 8 * (l.region0 + kVWaves * l.region);
    return l;
}

// LDS of a CU, which one block may have all of, and the kernel's own variables
// in it, with room to spare.
constexpr int kVLds = 160 * 1024, kVStatic = 256;

// The most that any robot, slot count and limit of a call asks for (72,768
// bytes, of 64 spheres in 3-D): every call's block fits.
constexpr int val_lds_most()
{
    ValDev v = {};
    int most = 0;
    auto take = [&](int kind, int D, int L, int dof) {
        v.kind = kind;
        v.D = D;
        v.L = L;
        v.vstride = 2 * dof + 3;
        for (v.B = 1; v.B <= (int)(sizeof(VRobot::rad) / sizeof(double)); ++v.B) {
            v.M = kVTile;
            const int n = val_lds(v, kValMaxActive).bytes;
            if (n > most) most = n;
        }
    };
    take(RGG_SE2, 2, 0, 3);
    take(RGG_SE3, 3, 0, 7);
    for (int L = 1; L <= (int)(sizeof(VRobot::len) / sizeof(double)); ++L) take(RGG_PLANAR_ARM, 2, L, L);
    return most;
}
static_assert(val_lds_most() == 72768 && val_lds_most() + kVStatic <= kVLds, "a validation block fits a CU");

// What one wavefront works on.
struct ValCtx {
    const ValDev &v;
    const ValLds &l;
    const double *rob;   // LDS: the robot and the resident boxes
    double *sd;          // LDS: this wavefront's region as doubles
    int32_t *si;         // the same as words
    int32_t *hit;        // LDS: smallest key of a colliding point of the step
    uint32_t *flag;      // LDS: bit k: child k of the chunk is not free
    unsigned long long *keep;   // LDS: boxes of each listed page that the next level's tests can reach
    int n_cand;          // present boxes near the edge
    bool cull;           // this step's tests fill keep
};

// Rounds outward for the near tests.  A lower bound above binary32's range, or
// an upper one below it, becomes NaN, which meets no box: no box lies out
// there (boxes are at most 1e30 in size).
__device__ inline float f32_below(double x) { return (float)x - fabsf((float)x) * 0x1p-22f - 0x1p-140f; }
__device__ inline float f32_above(double x) { return (float)x + fabsf((float)x) * 0x1p-22f + 0x1p-140f; }

// The box around a segment from a to b widened by R, and far beyond rounding:
// what lies outside it is farther than R from the segment.
__device__ inline double below(double a, double b, double R)
{
    const double mn = a < b ? a : b;
    return mn - (R * 1.000001 + 1e-9 * (1.0 + fabs(mn)));
}
__device__ inline double above(double a, double b, double R)
{
    const double mx = a < b ? b : a;
    return mx + (R * 1.000001 + 1e-9 * (1.0 + fabs(mx)));
}

// Binary32 boxes, 2 D floats each: a float4 in 2-D, three (lo, hi) pairs in
// 3-D.
template <int D>
__device__ __forceinline__ void put_box32(double *at, int k, const float *lo, const float *hi)
{
    if constexpr (D == 2) {
        reinterpret_cast<float4 *>(at)[k] = make_float4(lo[0], lo[1], hi[0], hi[1]);
    } else {
        float2 *g = reinterpret_cast<float2 *>(at) + 3 * k;
#pragma unroll
        for (int d = 0; d < D; ++d) g[d] = make_float2(lo[d], hi[d]);
    }
}

template <int D>
__device__ __forceinline__ bool meets32(const double *at, int k, const float *clo, const float *chi)
{
    if constexpr (D == 2) {
        const float4 q = reinterpret_cast<const float4 *>(at)[k];
        return (q.x <= chi[0]) & (q.y <= chi[1]) & (q.z >= clo[0]) & (q.w >= clo[1]);
    } else {
        const float2 *g = reinterpret_cast<const float2 *>(at) + 3 * k;
        bool r = true;
#pragma unroll
        for (int d = 0; d < D; ++d) {
            const float2 q = g[d];
            r = r & (q.x <= chi[d]) & (q.y >= clo[d]);
        }
        return r;
    }
}

// A resident box rounded outward; an ABSENT one (lo > hi on some axis) becomes
// one that meets nothing.
template <int D>
__device__ __forceinline__ void outward(const rgg_box &b, float *lo, float *hi)
{
    bool there = true;
#pragma unroll
    for (int d = 0; d < D; ++d) {
        there = there && b.lo[d] <= b.hi[d];
        lo[d] = f32_below(b.lo[d]);
        hi[d] = f32_above(b.hi[d]);
    }
    if (!there) lo[0] = NAN;
}

// Lists the slots of the present boxes that meet [clo, chi], in slot order from
// the lo_rank-th on, kVList at most; returns the number of all of them.
template <int D>
__device__ __forceinline__ int list_candidates(const ValCtx &x, const float *clo, const float *chi, int lo_rank)
{
    const int lane = threadIdx.x & 63;
    const int M = (int)x.v.M;
    const bool tiled = M <= kVTile;
    uint16_t *list = reinterpret_cast<uint16_t *>(x.sd + x.l.list);
    int base = 0;
    for (int s0 = 0; s0 < M; s0 += 64) {
        const int s = min(s0 + lane, M - 1);
        bool cand;
        if (tiled) {
            cand = meets32<D>(x.rob + x.l.tile, s, clo, chi);
        } else {
            float lo[D], hi[D];
            outward<D>(x.v.resident[s], lo, hi);
            cand = true;
#pragma unroll
            for (int d = 0; d < D; ++d) cand = cand & (lo[d] <= chi[d]) & (hi[d] >= clo[d]);
        }
        cand = cand && s0 + lane < M;
        const unsigned long long bal = __ballot(cand);
        const int rank = base + __popcll(bal & ((1ull << lane) - 1ull)) - lo_rank;
        if (cand && rank >= 0 && rank < kVList) list[rank] = (uint16_t)s;
        base += __popcll(bal);
    }
    wave_sync();
    return base;
}

// Puts the listed boxes l0 .. l0 + n (n <= kValBoxes) into LDS: the exact
// boxes, and their outward-rounded binary32 copies for the near tests.
template <int D>
__device__ __forceinline__ void stage_page(const ValCtx &x, int l0, int n)
{
    const int lane = threadIdx.x & 63;
    if (lane < n) {
        const uint16_t *list = reinterpret_cast<const uint16_t *>(x.sd + x.l.list);
        const rgg_box &b = x.v.resident[list[l0 + lane]];
        double *dst = x.sd + x.l.box + lane * 2 * D;
        float lo[D], hi[D];
        outward<D>(b, lo, hi);
#pragma unroll
        for (int d = 0; d < D; ++d) {
            dst[d] = b.lo[d];
            dst[D + d] = b.hi[d];
        }
        put_box32<D>(x.sd + x.l.box32, lane, lo, hi);
    }
    wave_sync();
}

// The sphere centres of nc configurations, t(q) the parameter of the q-th, in
// the build's expression order: at cen[(q B + i) D].  What the spheres of a
// configuration share is computed once, one lane each: the sine and cosine of
// every joint angle (arm) or of the heading, the two slerp weights (SE3), then
// the arm's joint positions.
template <int D, typename T>
__device__ __forceinline__ void centres(const ValCtx &x, int nc, T &&t_of)
{
    const ValDev &v = x.v;
    const int lane = threadIdx.x & 63, B = v.B, dof = v.dof;
    const double *mot = x.sd + x.l.mot, *a = mot, *b = mot + dof, *pos = x.rob + x.l.pos;
    double *fk = x.sd + x.l.fk, *cen = x.sd + x.l.cen;
    if (v.kind == RGG_PLANAR_ARM) {
        const int L = v.L, W = x.l.fkw;
        for (int w = lane; w < nc * L; w += 64) {
            const int q = w / L, m = w - q * L;
            const double t = t_of(q);
            double phi = a[0] + t * (b[0] - a[0]);
#pragma unroll 4
            for (int k = 1; k <= m; ++k) phi = phi + (a[k] + t * (b[k] - a[k]));
            double sn, cs;
            vsincos(phi, &sn, &cs);
            fk[q * W + m] = cs;
            fk[q * W + L + m] = sn;
        }
        wave_sync();
        const double *len = x.rob + x.l.len;
        for (int w = lane; w < nc * L; w += 64) {
            const int q = w / L, m = w - q * L;
            double jx = v.base[0], jy = v.base[1];
#pragma unroll 4
            for (int k = 0; k < m; ++k) {
                jx = jx + len[k] * fk[q * W + k];
                jy = jy + len[k] * fk[q * W + L + k];
            }
            fk[q * W + 2 * L + m] = jx;
            fk[q * W + 3 * L + m] = jy;
        }
        wave_sync();
        const int32_t *link = reinterpret_cast<const int32_t *>(x.rob) + x.l.link;
        for (int w = lane; w < nc * B; w += 64) {
            const int q = w / B, i = w - q * B, m = link[i];
            const double *f = fk + q * W + m;
            cen[w * D] = f[2 * L] + pos[i] * f[0];
            cen[w * D + 1] = f[3 * L] + pos[i] * f[L];
        }
    } else if (v.kind == RGG_SE2) {
        for (int q = lane; q < nc; q += 64) {
            double sn, cs;
            vsincos(a[2] + t_of(q) * mot[2 * dof], &sn, &cs);
            fk[2 * q] = cs;
            fk[2 * q + 1] = sn;
        }
        wave_sync();
        for (int w = lane; w < nc * B; w += 64) {
            const int q = w / B, i = w - q * B;
            const double t = t_of(q), co = fk[2 * q], s = fk[2 * q + 1];
            const double q0 = a[0] + t * (b[0] - a[0]);
            const double q1 = a[1] + t * (b[1] - a[1]);
            const double ox = pos[2 * i], oy = pos[2 * i + 1];
            cen[w * D] = q0 + (co * ox - s * oy);
            cen[w * D + 1] = q1 + (s * ox + co * oy);
        }
    } else if constexpr (D == 3) {
        const double half = mot[2 * dof + 1], sh = mot[2 * dof + 2];
        const bool turn = !(sh < 1e-12);
        if (turn) {
            for (int w = lane; w < 2 * nc; w += 64) {
                const double t = t_of(w >> 1);
                double sn, cs;
                vsincos((w & 1 ? t : 1.0 - t) * half, &sn, &cs);
                fk[w] = sn / sh;
            }
        }
        wave_sync();
        for (int w = lane; w < nc * B; w += 64) {
            const int q = w / B, i = w - q * B;
            const double t = t_of(q);
            const double q0 = a[0] + t * (b[0] - a[0]);
            const double q1 = a[1] + t * (b[1] - a[1]);
            const double q2 = a[2] + t * (b[2] - a[2]);
            double qw = a[3], ux = a[4], uy = a[5], uz = a[6];
            if (turn) {
                const double wa = fk[2 * q], wb = fk[2 * q + 1];
                qw = wa * a[3] + wb * b[3];
                ux = wa * a[4] + wb * b[4];
                uy = wa * a[5] + wb * b[5];
                uz = wa * a[6] + wb * b[6];
            }
            const double vx = pos[3 * i], vy = pos[3 * i + 1], vz = pos[3 * i + 2];
            const double tx = 2.0 * (uy * vz - uz * vy);
            const double ty = 2.0 * (uz * vx - ux * vz);
            const double tz = 2.0 * (ux * vy - uy * vx);
            const double rx = (vx + qw * tx) + (uy * tz - uz * ty);
            const double ry = (vy + qw * ty) + (uz * tx - ux * tz);
            const double rz = (vz + qw * tz) + (ux * ty - uy * tx);
            cen[w * D] = q0 + rx;
            cen[w * D + 1] = q1 + ry;
            cen[w * D + 2] = q2 + rz;
        }
    }
    wave_sync();
}

// One step of the search over the staged configurations: a wavefront's tests
// of points (a sphere at a configuration against the boxes) and of capsules (a
// sphere's over a sub-interval).
// kFirst: configurations 0, 1, 2 are t = 0, 1/2, 1.  Points t = 0 (key 0),
// t = 1 (key 1), t = 1/2 (key 2); capsules of the two halves (flag bits 0, 1)
// and of the whole edge (bit 2).
// Otherwise interval c of the chunk has its start, midpoint and end at
// configurations 3c .. 3c + 2: the midpoint (key 2 act + 1) and the two
// children's capsules (bits 2c, 2c + 1).  wl is the children's length.
// *hit receives the smallest key whose point collides (kNoHit if none), *flag
// the capsules that are not free; the children's bits are not complete when a
// point collides, nor bit 2 when t = 0 or 1 does (they do not matter then),
// and no capsule is tested when `points_only`.
//
// A lane first marks the staged boxes that its test's own bounding box meets
// (widened far beyond rounding, so a box left out cannot meet the test), then
// runs the exact test on the marked ones: the wavefront runs the expensive
// capsule test as often as the lane with the most near boxes needs it, not
// once for every box that any lane is near.
template <int D, bool kFirst>
__device__ __forceinline__ void run_tests(const ValCtx &x, const float *elo, const float *ehi, int n_int, double wl,
                                          const int32_t *act, bool points_only)
{
    constexpr int kParts = kFirst ? 6 : 3;
    const int lane = threadIdx.x & 63, B = x.v.B;
    const double *cen = x.sd + x.l.cen, *rad = x.rob + x.l.rad, *del = x.sd + x.l.del;
    if (lane == 0) {
        *x.hit = kNoHit;
        *x.flag = 0u;
    }
    wave_sync();
    const int tasks = n_int * kParts * B;
    for (int p0 = 0; p0 < x.n_cand; p0 += kValBoxes) {
        const int nb = min(kValBoxes, x.n_cand - p0);
        // one page stays staged; more come and go in every step
        if (x.n_cand > kValBoxes) {
            if (x.n_cand > kVList && p0 % kVList == 0) list_candidates<D>(x, elo, ehi, p0);
            stage_page<D>(x, p0 % kVList, nb);
        }
        // few tasks: several lanes per task, each taking every G-th box
        int G = tasks < 64 ? 64 / tasks : 1;
        if (G > nb) G = nb;
        for (int w0 = 0; w0 < tasks * G; w0 += 64) {
            const int w = w0 + lane;
            const int task = G == 1 ? w : w / G, grp = G == 1 ? 0 : w - task * G;
            const int r = task / B, i = task - r * B;
            const int c = kFirst ? 0 : r / kParts, part = kFirst ? r : r - kParts * c;
            const bool point = kFirst ? part < 3 : part == 0;
            int qa, qb;
            if (kFirst) {
                qa = part == 1 ? 2 : (part == 2 || part == 4 ? 1 : 0);
                qb = part == 3 ? 1 : 2;
            } else {
                qa = 3 * c + (part == 1 ? 0 : 1);
                qb = 3 * c + (part == 2 ? 2 : 1);
            }
            if (point) qb = qa;
            const double cw = kFirst && part == 5 ? 1.0 : wl;
            Capsule64<D> cap;
            unsigned long long m = 0, far = 0;
            double R = 0.0;
            if (w < tasks * G && (point || !points_only)) {
                R = point ? rad[i] : rad[i] + del[i] * (cw * cw);
                float clo[D], chi[D];
#pragma unroll
                for (int d = 0; d < D; ++d) {
                    cap.A[d] = cen[(qa * B + i) * D + d];
                    cap.B[d] = cen[(qb * B + i) * D + d];
                    clo[d] = f32_below(below(cap.A[d], cap.B[d], R));
                    chi[d] = f32_above(above(cap.A[d], cap.B[d], R));
                }
                const double *b32 = x.sd + x.l.box32;
                if (x.cull && !point && !(kFirst && part == 5)) {
                    // this capsule's motion stays within delta of its chord,
                    // its parts' tests within another r + delta of that
                    const double W = R + del[i] * (cw * cw);
                    float flo[D], fhi[D];
#pragma unroll
                    for (int d = 0; d < D; ++d) {
                        flo[d] = f32_below(below(cap.A[d], cap.B[d], W));
                        fhi[d] = f32_above(above(cap.A[d], cap.B[d], W));
                    }
                    int b = grp;
                    for (; b + 3 * G < nb; b += 4 * G) {
                        bool nr[4];
#pragma unroll
                        for (int u = 0; u < 4; ++u) nr[u] = meets32<D>(b32, b + u * G, flo, fhi);
#pragma unroll
                        for (int u = 0; u < 4; ++u) far |= (unsigned long long)nr[u] << (b + u * G);
                    }
                    for (; b < nb; b += G) far |= (unsigned long long)meets32<D>(b32, b, flo, fhi) << b;
                }
                int b = grp;
                for (; b + 7 * G < nb; b += 8 * G) {
                    bool nr[8];
#pragma unroll
                    for (int u = 0; u < 8; ++u) nr[u] = meets32<D>(b32, b + u * G, clo, chi);
                    if (G == 1) {
                        uint32_t byte = 0;
#pragma unroll
                        for (int u = 0; u < 8; ++u) byte |= nr[u] ? 1u << u : 0u;
                        m |= (unsigned long long)byte << b;
                    } else {
#pragma unroll
                        for (int u = 0; u < 8; ++u) m |= (unsigned long long)nr[u] << (b + u * G);
                    }
                }
                for (; b < nb; b += G) m |= (unsigned long long)meets32<D>(b32, b, clo, chi) << b;
            }
            if (x.cull) {
                for (int o = 32; o > 0; o >>= 1) far |= __shfl_xor(far, o);
                if (lane == 0) x.keep[p0 / kValBoxes] |= far;
            }
            if (point) {
                while (m) {
                    const int b = __ffsll(m) - 1;
                    m &= m - 1;
                    const double *bx = x.sd + x.l.box + b * 2 * D;
                    if (point_box64<D>(cap.A, bx, bx + D) <= R * R) {
                        atomicMin(x.hit, kFirst ? part : 2 * act[c] + 1);
                        m = 0;
                    }
                }
            }
            wave_sync();
            // a colliding point ends the search: the children do not matter
            const int h = *x.hit;
            const bool skip = points_only || (kFirst ? h < 2 || (h == 2 && part < 5) : h != kNoHit);
            const uint32_t bit = kFirst ? 1u << (part >= 3 ? part - 3 : 0) : 1u << (2 * c + (part == 2 ? 1 : 0));
            if (skip || point) m = 0;
            if (__ballot(m != 0)) {
                cap.set(R);
                while (m) {
                    const int b = __ffsll(m) - 1;
                    m &= m - 1;
                    const double *bx = x.sd + x.l.box + b * 2 * D;
                    if (cap.meets(bx, bx + D)) {
                        atomicOr(x.flag, bit);
                        m = 0;
                    }
                    // another sphere of the same capsule set may have met a box
                    if (__hip_atomic_load(x.flag, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP) & bit) m = 0;
                }
            }
        }
    }
    wave_sync();
}

// After a level whose tests filled x.keep: the candidates that no later test
// can reach leave the list.
template <int D>
__device__ __forceinline__ void drop_candidates(ValCtx &x)
{
    const int lane = threadIdx.x & 63;
    uint16_t *list = reinterpret_cast<uint16_t *>(x.sd + x.l.list);
    wave_sync();
    int n = 0;
    for (int p0 = 0; p0 < x.n_cand; p0 += kValBoxes) {
        const unsigned long long k = x.keep[p0 / kValBoxes];
        const uint16_t s = list[p0 + lane < x.n_cand ? p0 + lane : p0];
        wave_sync();
        if ((k >> lane) & 1ull) list[n + __popcll(k & ((1ull << lane) - 1ull))] = s;   // moves down only
        n += __popcll(k);
    }
    wave_sync();
    if (n < x.n_cand) {
        x.n_cand = n;
        if (n <= kValBoxes) stage_page<D>(x, 0, n);
    }
}

// The candidate region of edge e: its chords widened by r_i + 2 delta_i, plus
// a margin, rounded outward.  Its motion and chord deviations go to LDS.
template <int D>
__device__ __forceinline__ void load_edge(const ValCtx &x, int64_t e, float *elo, float *ehi)
{
    const ValDev &v = x.v;
    const int lane = threadIdx.x & 63, B = v.B;
    const int i = lane < B ? lane : 0;   // idle lanes repeat sphere 0
    for (int k = lane; k < v.vstride; k += 64) x.sd[x.l.mot + k] = v.motion[e * v.vstride + k];
    const double *cp = v.cap64 + e * (2 * D + 1) * B;
    const double dl = v.delta[e * B + i];
    if (lane < B) x.sd[x.l.del + lane] = dl;
    const double wd = cp[2 * D * B + i] + dl;
#pragma unroll
    for (int d = 0; d < D; ++d) {
        const double A = cp[d * B + i], Bv = cp[(D + d) * B + i];
        const double lo = (A < Bv ? A : Bv) - wd, hi = (A < Bv ? Bv : A) + wd;
        elo[d] = f32_below(lo - 1e-6 * (1.0 + fabs(lo)));
        ehi[d] = f32_above(hi + 1e-6 * (1.0 + fabs(hi)));
    }
    for (int o = 1; o < B; o <<= 1) {
#pragma unroll
        for (int d = 0; d < D; ++d) {
            elo[d] = fminf(elo[d], __shfl_xor(elo[d], o));
            ehi[d] = fmaxf(ehi[d], __shfl_xor(ehi[d], o));
        }
    }
#pragma unroll
    for (int d = 0; d < D; ++d) {
        elo[d] = __shfl(elo[d], 0);   // the first lanes hold every sphere's
        ehi[d] = __shfl(ehi[d], 0);
    }
}

// Whether a step looks for candidates to drop: from where a second bounding
// test per box costs less than the boxes it spares the later levels (most
// searches end after a level or two).  The whole list has to be known.
__device__ inline bool culls(const ValCtx &x) { return x.n_cand >= kVCull && x.n_cand <= kVList; }

// The search over an edge's motion; its region, boxes and motion are staged.
template <int D>
__device__ __forceinline__ void search(ValCtx &x, const float *elo, const float *ehi, int max_level,
                                       int max_active, uint8_t *out, int32_t *out_level, double *out_t)
{
    const int lane = threadIdx.x & 63;
    *out = kFree;
    *out_level = 0;
    *out_t = NAN;
    if (x.n_cand == 0) return;
    // t = 0, then t = 1, then the whole edge's capsules, and with them the
    // first level's midpoint and halves
    if (lane < kVList / kValBoxes) x.keep[lane] = 0ull;
    x.cull = culls(x);
    centres<D>(x, 3, [](int q) { return ldexp((double)q, -1); });
    run_tests<D, true>(x, elo, ehi, 1, 0.5, nullptr, false);
    int best = *x.hit;
    uint32_t fl = *x.flag;
    if (best < 2) {
        *out = kCollides;
        *out_t = (double)best;
        return;
    }
    if (!(fl & 4u)) return;
    int32_t *act = x.si + x.l.act, *nxt = x.si + x.l.nxt;
    int na = 1;
    if (lane == 0) act[0] = 0;
    if (best == 2) best = 1;   // the midpoint's key at level 0
    wave_sync();
    for (int l = 0; l < max_level; ++l) {
        *out_level = l;
        if (na > max_active) {
            *out = kUnresolved;
            return;
        }
        const double wl = ldexp(1.0, -(l + 1));
        int nn = 0;
        if (l > 0 && x.cull) {
            drop_candidates<D>(x);
            if (lane < kVList / kValBoxes) x.keep[lane] = 0ull;
            x.cull = culls(x);
        }
        for (int c0 = 0; c0 < na; c0 += x.l.chunk) {
            const int n_int = min(x.l.chunk, na - c0);
            const int32_t *ac = act + c0;
            if (l > 0) {
                centres<D>(x, 3 * n_int, [&](int q) {
                    const int c = q / 3;
                    return ldexp((double)(2 * ac[c] + (q - 3 * c)), -(l + 1));
                });
                run_tests<D, false>(x, elo, ehi, n_int, wl, ac, best != kNoHit);
                best = min(best, *x.hit);
                fl = *x.flag;
            }
            // the children that are not free, in order
            const bool open = lane < 2 * n_int && ((fl >> lane) & 1u);
            const unsigned long long bal = __ballot(open);
            const int at = nn + __popcll(bal & ((1ull << lane) - 1ull));
            if (open && at < max_active) nxt[at] = 2 * ac[lane >> 1] + (lane & 1);
            nn += __popcll(bal);
            wave_sync();
        }
        *out_level = l + 1;
        if (best != kNoHit) {
            *out = kCollides;
            *out_t = ldexp((double)best, -(l + 1));
            return;
        }
        if (nn == 0) return;   // FREE
        // more than max_active stops the search at the next level (or
        // after the last one) before the list is read again
        int32_t *const swap = act;
        act = nxt;
        nxt = swap;
        na = nn;
    }
    *out = kUnresolved;
}

// One wavefront per edge, four to a block.  The search is a chain of dependent
// binary64 phases per edge (10 us at the median, 30 to 60 for the deepest), so
// edges in flight matter more than threads per edge.  The grid is what the
// device holds at once, but no more than gives every wavefront an edge; each of
// these G blocks takes every G-th edge of the list, its wavefronts claiming
// them one at a time, so the robot and the resident boxes are staged once and a
// long search keeps one wavefront, not its block.
// What bounds it is the latency of the phases: on one update's gray lists,
//   arm, 13.9k edges:      535 us with each test's centres placed anew and
//     every box tested by every wavefront, 211 with a configuration's
//     kinematics computed once, 160 with claimed edges and binary32 near
//     tests, 117 with candidates dropped between levels (the deepest edges
//     held 120 boxes through nine levels);
//   spatial, 1.5k edges:   64, 46, 35, 32 us.
// The 3-D kernel needs 185 registers: at three blocks per CU it spills (32 us
// for 1,470 spatial edges against 31), the 2-D one does not (115 us for 13.9k
// arm edges, 123 at four).
constexpr int v_blocks_per_cu(int D) { return D == 3 ? 2 : 3; }

template <int D>
__global__ __launch_bounds__(kVT, v_blocks_per_cu(D)) void k_validate(ValDev v, ValLds l, const int64_t *ids, int64_t n,
                                                     const rgg_update_result *count, int max_level, int max_active,
                                                     uint8_t *verdict, int32_t *level, double *witness, uint8_t *labels)
{
    extern __shared__ __attribute__((aligned(16))) double sh[];
    __shared__ int32_t s_hit[kVWaves];
    __shared__ uint32_t s_flag[kVWaves];
    __shared__ unsigned long long s_keep[kVWaves][kVList / kValBoxes];
    __shared__ int32_t s_claim;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    int64_t nn = n;
    if (count) {
        const int64_t g = count->status == RGG_OK ? count->n_gray : 0;
        nn = g < n ? g : n;
    }
    // blocks beyond the list (the grid is sized for its capacity when the
    // count comes from the device) leave at once
    const int64_t full = (nn + kVWaves - 1) / kVWaves;
    const int64_t G = full < gridDim.x ? full : gridDim.x;
    if ((int64_t)blockIdx.x >= G) return;
    double *const mine = sh + l.region0 + wv * l.region;
    ValCtx x = {v, l, sh, mine, reinterpret_cast<int32_t *>(mine), &s_hit[wv], &s_flag[wv],
                s_keep[wv], 0, false};
    // the k-th edge of this block is list entry blockIdx + k G
    auto entry = [&](int k) { return (int64_t)blockIdx.x + k * G; };
    int64_t i = entry(wv);
    int64_t e = i < nn ? ids[i] : -1;
    {
        const VRobot &rb = *v.rob;
        const int per = v.kind == RGG_SE2 ? 2 : (v.kind == RGG_SE3 ? 3 : 1);
        if (tid < v.B * per) sh[l.pos + tid] = rb.pos[tid];
        if (tid < v.B) sh[l.rad + tid] = rb.rad[tid];
        if (tid < v.L) sh[l.len + tid] = rb.len[tid];
        if (tid < v.B) reinterpret_cast<int32_t *>(sh)[l.link + tid] = rb.link[tid];
        if (tid == 0) s_claim = kVWaves;
        if (v.M <= kVTile) {
            for (int k = tid; k < (int)v.M; k += kVT) {
                float lo[D], hi[D];
                outward<D>(v.resident[k], lo, hi);
                put_box32<D>(sh + l.tile, k, lo, hi);
            }
        }
    }
    __syncthreads();
    while (i < nn) {
        // the next claim and its edge id are under way during this search
        int k = 0;
        if (lane == 0) k = atomicAdd(&s_claim, 1);
        const int64_t i_next = entry(__builtin_amdgcn_readfirstlane(k));
        const int64_t e_next = i_next < nn ? ids[i_next] : -1;
        uint8_t out = RGG_VERDICT_BAD_ID;
        int32_t out_level = 0;
        double out_t = NAN;
        const bool ok = e >= 0 && e < v.E;
        if (ok) {
            float elo[D], ehi[D];
            load_edge<D>(x, e, elo, ehi);
            x.n_cand = v.M > 0 ? list_candidates<D>(x, elo, ehi, 0) : 0;
            if (x.n_cand <= kValBoxes) stage_page<D>(x, 0, x.n_cand);
            search<D>(x, elo, ehi, max_level, max_active, &out, &out_level, &out_t);
            wave_sync();
        }
        if (lane == 0) {
            if (verdict) verdict[i] = out;
            if (level) level[i] = out_level;
            if (witness) witness[i] = out_t;
            if (labels && ok) labels[e] = out == kFree ? (uint8_t)RGG_GREEN : (uint8_t)RGG_RED;
        }
        i = i_next;
        e = e_next;
    }
}

}  // namespace

hipError_t launch_validate(const ValDev &v, const int64_t *ids, int64_t n, const rgg_update_result *count,
                           int32_t max_level, int32_t max_active, uint8_t *verdict, int32_t *level,
                           double *witness, uint8_t *labels, hipStream_t s, hipEvent_t done)
{
    if (n <= 0) return done ? hipEventRecord(done, s) : hipSuccess;
    const ValLds l = val_lds(v, max_active);
    // the blocks that the device holds at once, by registers and by LDS
    const int64_t fit = kVLds / (l.bytes + kVStatic), most = v_blocks_per_cu(v.D);
    const int64_t held = (int64_t)v.n_cu * (fit > most ? most : fit);
    const int64_t full = (n + kVWaves - 1) / kVWaves;
    const int grid = (int)(full < held ? full : held);
    void *args[] = {(void *)&v,         (void *)&l,       (void *)&ids,     (void *)&n,     (void *)&count,   (void *)&max_level,
                    (void *)&max_active, (void *)&verdict, (void *)&level, (void *)&witness, (void *)&labels};
    return launch_marked(v.D == 3 ? (void *)k_validate<3> : (void *)k_validate<2>, dim3(grid), dim3(kVT), args, s,
                         done, (unsigned)l.bytes);
}

}  // namespace rgg
