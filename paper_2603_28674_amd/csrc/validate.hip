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
// One wavefront (a 64-thread block) validates one listed edge at a time (grid-stride
// over the list).  Its present boxes near the edge are staged in LDS: a box
// can matter only if it meets the box around the edge's chords widened by
// r_i + 2 delta_i (each sub-chord stays within delta_i of the edge's chord,
// each sub-capsule adds at most r_i + delta_i), plus a rounding margin.  More
// than kValBoxes such boxes are handled in pages.
#include <hip/hip_runtime.h>
#include <math.h>

#include "predicates64.h"
#include "rgg_device.h"

namespace rgg {

namespace {

constexpr int kVT = 64;            // threads per block
static_assert(kValBoxes <= 64, "a lane marks a page's boxes in 64 bits");
constexpr int kVGrid = 16384;      // blocks at most (the hardware balances them)
constexpr int kNoHit = 0x7fffffff;

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
// call (offsets in doubles, then in 32-bit words after them): a planar robot
// of few spheres then leaves room for more edges in flight.
struct ValLds {
    int mot, del, pos, rad, len, box, cen, fk;   // doubles
    int link, act, nxt;                          // 32-bit words
    int bytes;
    int chunk;       // intervals refined together
    int fkw;         // doubles per configuration at fk
    int box_n;       // candidate boxes per page
};

constexpr int kVChunkMax = 8;        // intervals per chunk at most (16 child flags in one word)
constexpr int kVCenDoubles = 768;    // sphere centres of a chunk (more when one interval needs it)

inline ValLds val_lds(const ValDev &v, int max_active)
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
    l.box_n = (int)(v.M < kValBoxes ? (v.M > 0 ? v.M : 1) : kValBoxes);
    int d = 0;
    auto take = [&](int n) {
        const int at = d;
        d += n;
        return at;
    };
    l.mot = take(v.vstride);
    l.del = take(v.B);
    l.pos = take(v.B * (v.kind == RGG_SE2 ? 2 : (v.kind == RGG_SE3 ? 3 : 1)));
    l.rad = take(v.B);
    l.len = take(v.L);
    l.box = take(l.box_n * 2 * v.D);
    l.cen = take(3 * l.chunk * v.B * v.D);
    l.fk = take(3 * l.chunk * l.fkw);
    d *= 2;
    l.link = take(v.kind == RGG_PLANAR_ARM ? v.B : 0);
    l.act = take(max_active);
    l.nxt = take(max_active);
    l.bytes = 4 * d;
    return l;
}

// What one wavefront works on.
struct ValCtx {
    const ValDev &v;
    const ValLds &l;
    double *sd;          // LDS as doubles
    int32_t *si;         // the same as words
    int32_t *hit;        // LDS: smallest key of a colliding point of the step
    uint32_t *flag;      // LDS: bit k: child k of the chunk is not free
    int n_cand;          // present boxes near the edge
};

// Stages the candidate boxes [page * box_n, ...) in LDS (lo[D], hi[D], in slot
// order); returns the number of candidates of all pages.  Four slots per lane
// are requested together.
template <int D>
__device__ __forceinline__ int gather_page(const ValCtx &x, const double *elo, const double *ehi, int page)
{
    constexpr int kU = 4;
    const int lane = threadIdx.x;
    const int lo_rank = page * x.l.box_n;
    const int M = (int)x.v.M;
    int base = 0;
    for (int s0 = 0; s0 < M; s0 += 64 * kU) {
        double lo[kU][D], hi[kU][D];
#pragma unroll
        for (int u = 0; u < kU; ++u) {
            const int s = s0 + u * 64 + lane;
            const rgg_box &b = x.v.resident[s < M ? s : M - 1];
#pragma unroll
            for (int k = 0; k < D; ++k) {
                lo[u][k] = b.lo[k];
                hi[u][k] = b.hi[k];
            }
        }
#pragma unroll
        for (int u = 0; u < kU; ++u) {
            bool cand = s0 + u * 64 + lane < M;
#pragma unroll
            for (int k = 0; k < D; ++k)
                cand = cand && lo[u][k] <= hi[u][k] && lo[u][k] <= ehi[k] && hi[u][k] >= elo[k];
            const unsigned long long bal = __ballot(cand);
            const int rank = base + __popcll(bal & ((1ull << lane) - 1ull)) - lo_rank;
            if (cand && rank >= 0 && rank < x.l.box_n) {
                double *dst = x.sd + x.l.box + rank * 2 * D;
#pragma unroll
                for (int k = 0; k < D; ++k) {
                    dst[k] = lo[u][k];
                    dst[D + k] = hi[u][k];
                }
            }
            base += __popcll(bal);
        }
    }
    __syncthreads();
    return base;
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
    const int lane = threadIdx.x, B = v.B, dof = v.dof;
    const double *mot = x.sd + x.l.mot, *a = mot, *b = mot + dof, *pos = x.sd + x.l.pos;
    double *fk = x.sd + x.l.fk, *cen = x.sd + x.l.cen;
    if (v.kind == RGG_PLANAR_ARM) {
        const int L = v.L, W = x.l.fkw;
        for (int w = lane; w < nc * L; w += 64) {
            const int q = w / L, m = w - q * L;
            const double t = t_of(q);
            double phi = a[0] + t * (b[0] - a[0]);
            for (int k = 1; k <= m; ++k) phi = phi + (a[k] + t * (b[k] - a[k]));
            double sn, cs;
            vsincos(phi, &sn, &cs);
            fk[q * W + m] = cs;
            fk[q * W + L + m] = sn;
        }
        __syncthreads();
        const double *len = x.sd + x.l.len;
        for (int w = lane; w < nc * L; w += 64) {
            const int q = w / L, m = w - q * L;
            double jx = v.base[0], jy = v.base[1];
            for (int k = 0; k < m; ++k) {
                jx = jx + len[k] * fk[q * W + k];
                jy = jy + len[k] * fk[q * W + L + k];
            }
            fk[q * W + 2 * L + m] = jx;
            fk[q * W + 3 * L + m] = jy;
        }
        __syncthreads();
        const int32_t *link = x.si + x.l.link;
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
        __syncthreads();
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
        __syncthreads();
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
    __syncthreads();
}

// One step of the search over the staged configurations: three tests per
// interval and sphere.  kLevel0: the points t = 0 (key 0) and t = 1 (key 1)
// and the whole edge's capsule (flag bit 0), configurations 0, 1, 2 being
// t = 0, 1/2, 1.  Otherwise interval c of the chunk has its start, midpoint
// and end at configurations 3c .. 3c + 2: the midpoint (key 2 act + 1) and the
// two children's capsules (flag bits 2c, 2c + 1), wl the children's length.
// *hit receives the smallest key whose point collides (kNoHit if none), *flag
// the children that are not free (not to be used when a point collides; not
// computed when `points_only`).
//
// A lane first marks the staged boxes that its test's own bounding box meets
// (widened far beyond rounding, so a box left out cannot meet the test), then
// runs the exact test on the marked ones: the wavefront runs the expensive
// segment-box minimum as often as the lane with the most near boxes needs it,
// not once for every box that any lane is near.
template <int D, bool kLevel0>
__device__ __forceinline__ void run_tests(const ValCtx &x, const double *elo, const double *ehi, int n_int, double wl,
                                          const int32_t *act, bool points_only)
{
    const int lane = threadIdx.x, B = x.v.B;
    const double *cen = x.sd + x.l.cen, *rad = x.sd + x.l.rad, *del = x.sd + x.l.del;
    if (lane == 0) {
        *x.hit = kNoHit;
        *x.flag = 0u;
    }
    __syncthreads();
    const int tasks = n_int * 3 * B;
    const int n_pages = (x.n_cand + x.l.box_n - 1) / x.l.box_n;
    for (int p = 0; p < n_pages; ++p) {
        if (n_pages > 1) gather_page<D>(x, elo, ehi, p);
        const int nb = min(x.l.box_n, x.n_cand - p * x.l.box_n);
        // few tasks: several lanes per task, each taking every G-th box
        int G = tasks < 64 ? 64 / tasks : 1;
        if (G > nb) G = nb;
        for (int w0 = 0; w0 < tasks * G; w0 += 64) {
            const int w = w0 + lane;
            const int task = G == 1 ? w : w / G, grp = G == 1 ? 0 : w - task * G;
            const int r = task / B, i = task - r * B;
            const int c = r / 3, part = r - 3 * c;
            const bool live = w < tasks * G;
            const bool point = kLevel0 ? part < 2 : part == 0;
            const int qa = kLevel0 ? (part == 1 ? 2 : 0) : 3 * c + (part == 1 ? 0 : 1);
            const int qb = kLevel0 ? (part == 0 ? 0 : 2) : 3 * c + (part == 2 ? 2 : 1);
            double ca[D], cb[D], R = 0.0;
            unsigned long long m = 0;
            if (live && (point || !points_only)) {
                R = point ? rad[i] : rad[i] + del[i] * (wl * wl);
                double clo[D], chi[D];
#pragma unroll
                for (int d = 0; d < D; ++d) {
                    ca[d] = cen[(qa * B + i) * D + d];
                    cb[d] = cen[(qb * B + i) * D + d];
                    const double mn = ca[d] < cb[d] ? ca[d] : cb[d], mx = ca[d] < cb[d] ? cb[d] : ca[d];
                    clo[d] = mn - (R * 1.000001 + 1e-9 * (1.0 + fabs(mn)));
                    chi[d] = mx + (R * 1.000001 + 1e-9 * (1.0 + fabs(mx)));
                }
                for (int b = grp; b < nb; b += G) {
                    const double *bx = x.sd + x.l.box + b * 2 * D;
                    bool near = true;
#pragma unroll
                    for (int d = 0; d < D; ++d) near = near && bx[d] <= chi[d] && bx[D + d] >= clo[d];
                    m |= (unsigned long long)near << b;
                }
            }
            if (point) {
                while (m) {
                    const int b = __ffsll(m) - 1;
                    m &= m - 1;
                    const double *bx = x.sd + x.l.box + b * 2 * D;
                    if (point_box64<D>(ca, bx, bx + D) <= R * R) {
                        atomicMin(x.hit, kLevel0 ? part : 2 * act[c] + 1);
                        m = 0;
                    }
                }
            }
            __syncthreads();
            // a colliding point ends the search: the children do not matter
            if (*x.hit != kNoHit) points_only = true;
            if (points_only || point) m = 0;
            const uint32_t bit = kLevel0 ? 1u : 1u << (2 * c + part - 1);
            while (m) {
                const int b = __ffsll(m) - 1;
                m &= m - 1;
                const double *bx = x.sd + x.l.box + b * 2 * D;
                if (segbox64<D>(ca, cb, bx, bx + D) <= R * R) {
                    atomicOr(x.flag, bit);
                    m = 0;
                }
            }
        }
    }
    __syncthreads();
}

template <int D>
__device__ __forceinline__ void validate_one(ValCtx &x, int64_t e, int max_level, int max_active, uint8_t *verdict,
                                             int32_t *level, double *witness, uint8_t *labels)
{
    const ValDev &v = x.v;
    const int lane = threadIdx.x, B = v.B;
    // the edge's motion and chord deviations, and its capsules for the
    // candidate region: one round of loads
    for (int k = lane; k < v.vstride; k += 64) x.sd[x.l.mot + k] = v.motion[e * v.vstride + k];
    double elo[D], ehi[D];
    {
        // the chords widened by r_i + 2 delta_i, plus a margin
        const double *cp = v.cap64 + e * (2 * D + 1) * B;
        const double dl = lane < B ? v.delta[e * B + lane] : 0.0;
        if (lane < B) x.sd[x.l.del + lane] = dl;
        const double wd = lane < B ? cp[2 * D * B + lane] + dl : 0.0;
#pragma unroll
        for (int d = 0; d < D; ++d) {
            const double A = lane < B ? cp[d * B + lane] : 0.0, Bv = lane < B ? cp[(D + d) * B + lane] : 0.0;
            const double mn = A < Bv ? A : Bv, mx = A < Bv ? Bv : A;
            elo[d] = lane < B ? mn - wd : INFINITY;
            ehi[d] = lane < B ? mx + wd : -INFINITY;
        }
        for (int o = 1; o < B; o <<= 1) {
#pragma unroll
            for (int d = 0; d < D; ++d) {
                const double l2 = __shfl_xor(elo[d], o), h2 = __shfl_xor(ehi[d], o);
                elo[d] = l2 < elo[d] ? l2 : elo[d];
                ehi[d] = h2 > ehi[d] ? h2 : ehi[d];
            }
        }
#pragma unroll
        for (int d = 0; d < D; ++d) {
            const double lo = __shfl(elo[d], 0), hi = __shfl(ehi[d], 0);
            elo[d] = lo - 1e-6 * (1.0 + fabs(lo));
            ehi[d] = hi + 1e-6 * (1.0 + fabs(hi));
        }
    }
    x.n_cand = v.M > 0 ? gather_page<D>(x, elo, ehi, 0) : 0;

    uint8_t out = kUnresolved;
    int32_t out_level = 0;
    double out_t = NAN;
    do {
        // t = 0, then t = 1, and the whole edge's capsules; the first
        // interval's midpoint comes along
        if (x.n_cand == 0) {
            out = kFree;
            break;
        }
        centres<D>(x, 3, [](int q) { return ldexp((double)q, -1); });
        run_tests<D, true>(x, elo, ehi, 1, 1.0, nullptr, false);
        const int h0 = *x.hit;
        if (h0 != kNoHit) {
            out = kCollides;
            out_t = (double)h0;
            break;
        }
        if (!*x.flag) {
            out = kFree;
            break;
        }
        int na = 1;
        int32_t *act = x.si + x.l.act, *nxt = x.si + x.l.nxt;
        if (lane == 0) act[0] = 0;
        __syncthreads();
        bool done = false;
        for (int l = 0; l < max_level; ++l) {
            out_level = l;
            if (na > max_active) {
                out = kUnresolved;
                done = true;
                break;
            }
            const double wl = ldexp(1.0, -(l + 1));
            int best = kNoHit, nn = 0;
            for (int c0 = 0; c0 < na; c0 += x.l.chunk) {
                const int n_int = min(x.l.chunk, na - c0);
                const int32_t *ac = act + c0;
                if (l > 0)
                    centres<D>(x, 3 * n_int, [&](int q) {
                        const int c = q / 3;
                        return ldexp((double)(2 * ac[c] + (q - 3 * c)), -(l + 1));
                    });
                run_tests<D, false>(x, elo, ehi, n_int, wl, ac, best != kNoHit);
                best = min(best, *x.hit);
                // the children that are not free, in order
                const bool open = lane < 2 * n_int && ((*x.flag >> lane) & 1u);
                const unsigned long long bal = __ballot(open);
                const int at = nn + __popcll(bal & ((1ull << lane) - 1ull));
                if (open && at < max_active) nxt[at] = 2 * ac[lane >> 1] + (lane & 1);
                nn += __popcll(bal);
                __syncthreads();
            }
            if (best != kNoHit) {
                out = kCollides;
                out_level = l + 1;
                out_t = ldexp((double)best, -(l + 1));
                done = true;
                break;
            }
            out_level = l + 1;
            if (nn == 0) {
                out = kFree;
                done = true;
                break;
            }
            // more than max_active stops the search at the next level (or
            // after the last one) before the list is read again
            int32_t *const swap = act;
            act = nxt;
            nxt = swap;
            na = nn;
        }
        if (!done) {
            out = kUnresolved;
            out_level = max_level;
        }
    } while (false);
    __syncthreads();
    if (lane == 0) {
        if (verdict) verdict[0] = out;
        if (level) level[0] = out_level;
        if (witness) witness[0] = out_t;
        if (labels) labels[e] = out == kFree ? (uint8_t)RGG_GREEN : (uint8_t)RGG_RED;
    }
    __syncthreads();
}

// One wavefront per edge.  The search is a chain of dependent binary64 phases
// per edge, so edges in flight matter more than threads per edge.  A step
// used to place every sphere of every test from the joint angles anew (an
// arm's sphere on its last link took all seven sine-cosine pairs, 84 per
// configuration of a 21-sphere arm instead of 7); with the shared centres and
// the marked boxes the update + validation of the arm with 56k edges (14.6k of
// them gray) went from 606 to 289 us, of the spatial body with 116k edges
// (1.5k gray) from 148 to 119 us.
template <int D>
__global__ __launch_bounds__(kVT) __attribute__((amdgpu_waves_per_eu(4))) void k_validate(
    ValDev v, ValLds l, const int64_t *ids, int64_t n, const rgg_update_result *count, int max_level, int max_active,
    uint8_t *verdict, int32_t *level, double *witness, uint8_t *labels)
{
    extern __shared__ double sh[];
    __shared__ int32_t s_hit;
    __shared__ uint32_t s_flag;
    const int lane = threadIdx.x;
    int64_t nn = n;
    if (count) {
        const int64_t g = count->status == RGG_OK ? count->n_gray : 0;
        nn = g < n ? g : n;
    }
    // blocks beyond the list (the grid is sized for its capacity when the
    // count comes from the device) leave at once
    if ((int64_t)blockIdx.x >= nn) return;
    ValCtx x = {v, l, sh, reinterpret_cast<int32_t *>(sh), &s_hit, &s_flag, 0};
    {
        const VRobot &rb = *v.rob;
        const int per = v.kind == RGG_SE2 ? 2 : (v.kind == RGG_SE3 ? 3 : 1);
        for (int k = lane; k < v.B * per; k += 64) x.sd[l.pos + k] = rb.pos[k];
        if (lane < v.B) x.sd[l.rad + lane] = rb.rad[lane];
        if (lane < v.L) x.sd[l.len + lane] = rb.len[lane];
        if (v.kind == RGG_PLANAR_ARM && lane < v.B) x.si[l.link + lane] = rb.link[lane];
    }
    for (int64_t i = blockIdx.x; i < nn; i += gridDim.x) {
        const int64_t e = ids[i];
        if (e < 0 || e >= v.E) {
            if (lane == 0) {
                if (verdict) verdict[i] = RGG_VERDICT_BAD_ID;
                if (level) level[i] = 0;
                if (witness) witness[i] = NAN;
            }
            continue;
        }
        validate_one<D>(x, e, max_level, max_active, verdict ? verdict + i : nullptr, level ? level + i : nullptr,
                        witness ? witness + i : nullptr, labels);
    }
}

}  // namespace

hipError_t launch_validate(const ValDev &v, const int64_t *ids, int64_t n, const rgg_update_result *count,
                           int32_t max_level, int32_t max_active, uint8_t *verdict, int32_t *level,
                           double *witness, uint8_t *labels, hipStream_t s, hipEvent_t done)
{
    if (n <= 0) return done ? hipEventRecord(done, s) : hipSuccess;
    const int grid = (int)(n < kVGrid ? n : kVGrid);
    const ValLds l = val_lds(v, max_active);
    void *args[] = {(void *)&v,         (void *)&l,       (void *)&ids,     (void *)&n,     (void *)&count,   (void *)&max_level,
                    (void *)&max_active, (void *)&verdict, (void *)&level, (void *)&witness, (void *)&labels};
    return launch_marked(v.D == 3 ? (void *)k_validate<3> : (void *)k_validate<2>, dim3(grid), dim3(kVT), args, s,
                         done, (unsigned)l.bytes);
}

}  // namespace rgg
