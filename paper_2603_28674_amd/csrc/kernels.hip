// Update pipeline of librgg for gfx950 (wave64).
//
// One update = these kernels on one stream (or one graph):
//   k_diff      validate the old/new boxes against the resident slots, list
//               the changed (box, sign) entries in slot order, commit the
//               slots (Alg. 1: a moved obstacle's old and new poses); with
//               one grid cell it also hands out the fixed work items, with
//               several it activates every grid cell a changed box overlaps
//               and emits one work item per (cell, chunk of its edges)
//               (Sec. 4.3);
//   k_item32/64 one block per work item: pairs of the item's edges with the
//               changed boxes of the cell, outer test (per-sphere capsule vs
//               box), inner test (copies of the spheres whose capsule met),
//               counter update (Sec. 4.1 rule; Alg. 1's intersection lists
//               kept as counts).  Optionally (inline_rounds) the FP32 item
//               kernel tests only an item's first pair rounds and lists the
//               rest for
//   k_pairs     which cuts the listed pairs into equal shares, one per
//               block, and runs the same tests on them.  In the FP32 mode a
//               pair whose margin falls inside the rounding band is decided
//               in binary64 by the block that tested it;
//   k_labels    labels from the counters and the ordered gray list, in one
//               pass (k_count + k_write, the two-pass form, serve the label
//               queries and the batch).
// The *_batch kernels run the same stages for many roadmaps in one launch
// each, reading every roadmap's arguments from a request table.
//
// Binary64 code is compiled without FMA contraction and its sums run left to
// right from 0.0, so a re-test reproduces the definition's values exactly.
// Hot loops keep off single global counters: on MI355X device-scope atomics
// on one address serialise across the eight XCDs, so work lists are
// positional and statistics go to 256 rows shared through atomics.  The few
// single-address counters are k_labels' tickets (one per 4096-edge tile) and
// the batched item kernel's claims (one per item past two per block).
#include <hip/hip_ext.h>
#include <hip/hip_runtime.h>

#include <type_traits>

#include "predicates64.h"
#include "rgg_device.h"

namespace rgg {

namespace {

constexpr int kDiffBlock = 1024;
constexpr int kFewChunks = 4;      // items that one thread emits for a cell
constexpr int kBlock = 256;
constexpr int kWaves = kBlock / 64;
constexpr int kGrid = kStatBlocks; // blocks of the item kernels
constexpr int kBatchItemGrid = 1024;  // blocks of a batched item kernel: the blocks of the
                                      // FP32 kernel resident at once (4 per CU, 256 CUs)
constexpr int kBatchStatic = 2;       // items a batched item block takes before it claims
static_assert(kStatBlocks % 256 == 0, "statistics rows are folded 256 at a time");

enum : int { kMiss = 0, kHit = 1, kUnsure = 2, kOpen = 3 };

__device__ inline int lane_id() { return __lane_id(); }
__device__ inline uint64_t lanes_below() { return (1ull << lane_id()) - 1ull; }

__device__ inline void wave_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

__device__ inline unsigned long long wave_sum_u64(unsigned long long v)
{
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
    return v;
}

__device__ inline int wave_prefix(int v, int *total)
{
    // inclusive scan over the wavefront, returned exclusive
    const int lane = lane_id();
    int x = v;
    for (int o = 1; o < 64; o <<= 1) {
        int y = __shfl_up(x, o);
        if (lane >= o) x += y;
    }
    *total = __shfl(x, 63);
    return x - v;
}

__device__ inline float next_down(float f)
{
    uint32_t b = __float_as_uint(f);
    if (f > 0.0f) return __uint_as_float(b - 1u);
    if (f < 0.0f) return __uint_as_float(b + 1u);
    return -__uint_as_float(1u);
}

__device__ inline float round_down(double x)
{
    float f = (float)x;
    return (double)f > x ? next_down(f) : f;
}

__device__ inline float round_up(double x)
{
    float f = (float)x;
    return (double)f < x ? -next_down(-f) : f;
}

__device__ inline int32_t cell_of(double x, double org, double inv, int32_t n)
{
    // c is integral, so comparing its int32 value with n decides c >= n
    // exactly (and keeps n out of binary64 registers)
    double c = floor((x - org) * inv);
    if (c < 0.0) return -1;
    if (!(c < 2147483647.0)) return n;
    const int32_t ci = (int32_t)c;
    return ci >= n ? n : ci;
}

// ------------------------------------------------------------------------
// binary32 filter: the same quantities, any rounding; only a margin outside
// the band +-band_rel*s^2 is trusted (s bounds every coordinate of the pair)
// ------------------------------------------------------------------------

template <int D>
__device__ inline float point_box32(const float *c, const float *lo, const float *hi)
{
    float acc = 0.0f;
#pragma unroll
    for (int k = 0; k < D; ++k) {
        float g = fmaxf(fmaxf(lo[k] - c[k], 0.0f), c[k] - hi[k]);
        acc = __builtin_fmaf(g, g, acc);
    }
    return acc;
}

template <int D>
__device__ inline float seg_F32(const float *A, const float *d, float t, const float *lo, const float *hi)
{
    float acc = 0.0f;
#pragma unroll
    for (int k = 0; k < D; ++k) {
        float p = __builtin_fmaf(t, d[k], A[k]);
        float g = fmaxf(fmaxf(lo[k] - p, 0.0f), p - hi[k]);
        acc = __builtin_fmaf(g, g, acc);
    }
    return acc;
}

// `targ` receives the parameter of the value returned.  Scheduling barriers
// between the candidates keep one candidate's temporaries live at a time, so
// this binary32 filter stays small in registers.
template <int D>
__device__ inline float segbox32(const float *A, const float *Bp, const float *lo, const float *hi, float &targ)
{
    float d[D], inv[D];
#pragma unroll
    for (int k = 0; k < D; ++k) {
        d[k] = Bp[k] - A[k];
        inv[k] = d[k] != 0.0f ? __builtin_amdgcn_rcpf(d[k]) : 0.0f;
    }
    float tL = 0.0f, tR = 1.0f;
    auto take = [&](float t) {
        float g = 0.0f;
#pragma unroll
        for (int k = 0; k < D; ++k) {
            float p = __builtin_fmaf(t, d[k], A[k]);
            float ex = fminf(p - lo[k], 0.0f) + fmaxf(p - hi[k], 0.0f);
            g = __builtin_fmaf(d[k], ex, g);
        }
        tL = (g <= 0.0f && t > tL) ? t : tL;
        tR = (g >= 0.0f && t < tR) ? t : tR;
        __builtin_amdgcn_sched_barrier(0);
    };
    take(0.0f);
    take(1.0f);
#pragma unroll
    for (int k = 0; k < D; ++k) {
        // a crossing outside (0,1) (or of an axis the segment does not
        // move along) is replaced by t = 0, which repeats the first candidate
        float t1 = (lo[k] - A[k]) * inv[k];
        take(t1 > 0.0f && t1 < 1.0f ? t1 : 0.0f);
        float t2 = (hi[k] - A[k]) * inv[k];
        take(t2 > 0.0f && t2 < 1.0f ? t2 : 0.0f);
    }
    const float fL = seg_F32<D>(A, d, tL, lo, hi), fR = seg_F32<D>(A, d, tR, lo, hi);
    const float fmin = fminf(fL, fR);
    const float tmin = fL <= fR ? tL : tR;
    float tm = 0.5f * (tL + tR);
    float num = 0.0f, den = 0.0f;
#pragma unroll
    for (int k = 0; k < D; ++k) {
        float p = __builtin_fmaf(tm, d[k], A[k]);
        float b = p < lo[k] ? lo[k] : (p > hi[k] ? hi[k] : A[k]);
        float w = (p < lo[k] || p > hi[k]) ? d[k] : 0.0f;
        num = __builtin_fmaf(w, b - A[k], num);
        den = __builtin_fmaf(w, w, den);
    }
    float ts = den > 0.0f ? fminf(fmaxf(num * __builtin_amdgcn_rcpf(den), tL), tR) : tL;
    const float fs = seg_F32<D>(A, d, ts, lo, hi);
    targ = fs < fmin ? ts : tmin;
    return fminf(fmin, fs);
}

__device__ inline int classify_margin(float m, float band)
{
    return m < -band ? kHit : (m > band ? kMiss : kUnsure);
}

// ------------------------------------------------------------------------
// k_diff: validation, changed entries, commit
// ------------------------------------------------------------------------

__device__ inline bool box_ok(const rgg_box &b)
{
    for (int k = 0; k < 3; ++k)
        if (!(fabs(b.lo[k]) <= 1e30) || !(fabs(b.hi[k]) <= 1e30)) return false;
    return true;
}

__device__ inline bool same_box(const rgg_box &a, const rgg_box &b)
{
    bool s = true;
    for (int k = 0; k < 3; ++k)
        s = s && __double_as_longlong(a.lo[k]) == __double_as_longlong(b.lo[k]) &&
            __double_as_longlong(a.hi[k]) == __double_as_longlong(b.hi[k]);
    return s;
}

template <int D>
__device__ inline bool present(const rgg_box &b)
{
    bool p = true;
#pragma unroll
    for (int k = 0; k < 3; ++k) p = p && (k >= D || b.lo[k] <= b.hi[k]);
    return p;
}

// returns whether the box covers at least one grid cell (D is the
// roadmap's dimension, so the loop below is straight-line code)
template <int D>
__device__ bool write_entry(const RmDev &rm, int pos, const rgg_box &b, int sign)
{
    ChgEntry en;
    float s = 0.0f;
    bool empty = false;
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        if (k < D) {
            en.lo[k] = b.lo[k];
            en.hi[k] = b.hi[k];
            en.lo32[k] = round_down(b.lo[k]);
            en.hi32[k] = round_up(b.hi[k]);
            s = fmaxf(s, fmaxf(fabsf(en.lo32[k]), fabsf(en.hi32[k])));
            int32_t a = cell_of((double)en.lo32[k], rm.gorg[k], rm.ginv, rm.gdim[k]);
            int32_t z = cell_of((double)en.hi32[k], rm.gorg[k], rm.ginv, rm.gdim[k]);
            if (z < 0 || a > rm.gdim[k] - 1) empty = true;
            en.c0[k] = a < 0 ? 0 : a;
            en.c1[k] = z > rm.gdim[k] - 1 ? rm.gdim[k] - 1 : z;
        } else {
            en.lo[k] = en.hi[k] = 0.0;
            en.lo32[k] = en.hi32[k] = 0.0f;
            en.c0[k] = en.c1[k] = 0;
        }
    }
    if (empty) {
        en.c0[0] = 1;
        en.c1[0] = 0;
    }
    en.sbox = s;
    en.sign = sign;
    rm.chg[pos] = en;
    return !empty;
}

// Block-wide exclusive prefix over the kNW wavefronts of a block (64-bit
// values): returns this thread's prefix, *total the block's sum.
template <int kNW>
__device__ inline long long block_prefix64(long long v, long long *total, long long *wsum)
{
    const int lane = lane_id(), wv = (int)(threadIdx.x >> 6);
    long long x = v;
    for (int o = 1; o < 64; o <<= 1) {
        const long long y = __shfl_up(x, o);
        if (lane >= o) x += y;
    }
    __syncthreads();
    if (lane == 63) wsum[wv] = x;
    __syncthreads();
    long long off = 0, tot = 0;
    for (int w = 0; w < kNW; ++w) {
        off += w < wv ? wsum[w] : 0;
        tot += wsum[w];
    }
    *total = tot;
    return off + x - v;
}

// Grid roadmaps: the cells the n_chg changed entries cover are marked and
// each newly marked cell emits one work item per chunk of its edges (an
// empty cell one item, whose first chunk clears the mark).  An item names its
// slots of the cell lists, so an item block needs no look at the cell.  One block of
// kDiffBlock threads, right after the entries are written: the (entry,
// cell) pairs are dealt over the threads (a prefix over the entries' cell
// counts), so every mark of a pass is in flight at once, and the items go
// to positions from a block scan (one block per roadmap: no global counter).
__device__ __forceinline__ void activate_cells(const RmDev &rm, int n_chg)
{
    constexpr int kNW = kDiffBlock / 64;
    __shared__ long long s_cpre[kDiffBlock];
    __shared__ int s_rng[kDiffBlock][5];   // first cell (x, y, z), cells along x and y
    __shared__ long long s_w64[kNW];
    __shared__ int s_w32[kNW];
    __shared__ int s_items, s_nbig;
    __shared__ int4 s_big[kDiffBlock];     // cells of many chunks: cell, first slot, slots, position
    const int tid = threadIdx.x, lane = lane_id(), wv = tid >> 6;
    if (tid == 0) {
        s_items = 0;
        s_nbig = 0;
    }
    auto put = [&](int pos, int cell, int s0, int n, int h) {
        if (pos < rm.items_cap) rm.items[pos] = make_int4(s0 + h * rm.chunk, min(rm.chunk, n - h * rm.chunk), cell, h);
    };
    for (int q0 = 0; q0 < n_chg; q0 += kDiffBlock) {
        const int q = q0 + tid;
        long long cnt = 0;
        if (q < n_chg) {
            const ChgEntry &en = rm.chg[q];
            const int32_t nx = en.c1[0] - en.c0[0] + 1, ny = en.c1[1] - en.c0[1] + 1, nz = en.c1[2] - en.c0[2] + 1;
            if (nx > 0 && ny > 0 && nz > 0) cnt = (long long)nx * ny * nz;
            s_rng[tid][0] = en.c0[0];
            s_rng[tid][1] = en.c0[1];
            s_rng[tid][2] = en.c0[2];
            s_rng[tid][3] = nx;
            s_rng[tid][4] = ny;
        }
        long long tot;
        const long long pre = block_prefix64<kNW>(cnt, &tot, s_w64);
        s_cpre[tid] = pre;
        __syncthreads();
        const int ne = min(kDiffBlock, n_chg - q0);
        for (long long t0 = 0; t0 < tot; t0 += kDiffBlock) {
            const long long t = t0 + tid;
            int nch = 0, s0 = 0, n = 0;
            long long c = 0;
            if (t < tot) {
                // the entry holding pair t: the last j with s_cpre[j] <= t
                int lo = 0, hi = ne - 1;
                while (lo < hi) {
                    const int mid = (lo + hi + 1) >> 1;
                    if (s_cpre[mid] <= t) lo = mid;
                    else hi = mid - 1;
                }
                const long long k = t - s_cpre[lo];
                const int nx = s_rng[lo][3], ny = s_rng[lo][4];
                const int32_t x = s_rng[lo][0] + (int32_t)(k % nx);
                const int32_t y = s_rng[lo][1] + (int32_t)((k / nx) % ny);
                const int32_t z = s_rng[lo][2] + (int32_t)(k / ((long long)nx * ny));
                c = ((long long)z * rm.gdim[1] + y) * rm.gdim[0] + x;
                const uint32_t bit = 1u << (c & 31);
                s0 = rm.cell_start[c];
                n = rm.cell_start[c + 1] - s0;
                if (!(atomicOr(&rm.cell_bits[c >> 5], bit) & bit)) {
                    nch = n > 0 ? (n + rm.chunk - 1) / rm.chunk : 1;
                }
            }
            // positions of this pass's items
            int x = nch;
            for (int o = 1; o < 64; o <<= 1) {
                const int y = __shfl_up(x, o);
                if (lane >= o) x += y;
            }
            __syncthreads();
            if (lane == 63) s_w32[wv] = x;
            __syncthreads();
            int off = s_items, ntot = 0;
            for (int w = 0; w < kNW; ++w) {
                off += w < wv ? s_w32[w] : 0;
                ntot += s_w32[w];
            }
            const int pos = off + x - nch;
            // a cell's items one after another on its thread, but a cell of
            // many chunks (coarse grids over many edges) on a wavefront: an arm
            // with 56k edges in 9 cells took 23 us here with one thread each
            if (nch <= kFewChunks) {
                for (int h = 0; h < nch; ++h) put(pos + h, (int)c, s0, n, h);
            } else {
                s_big[atomicAdd(&s_nbig, 1)] = make_int4((int)c, s0, n, pos);
            }
            __syncthreads();
            for (int b = wv; b < s_nbig; b += kNW) {
                const int4 w = s_big[b];
                for (int h = lane; h * rm.chunk < w.z; h += 64) put(w.w + h, w.x, w.y, w.z, h);
            }
            __syncthreads();
            if (tid == 0) {
                s_items += ntot;
                s_nbig = 0;
            }
            __syncthreads();
        }
    }
    if (tid == 0) rm.ctl->n_items = s_items;
}

// One block: validates the update, writes the changed entries and commits
// the new boxes.  The block's first half takes the entry of a slot's old
// box, the second half that of its new box, so each thread writes at most
// one entry (the entry is a chain of binary64 roundings and cell indices,
// which one wavefront runs at its latency); a chunk of the update covers
// kDiffBlock / 2 slots, its old boxes' entries first.
// n_fixed: the number of fixed items that the item kernel will visit, 0 when a
// grid's cells have to be activated.
template <int D>
__device__ __forceinline__ void diff_body(const RmDev &rm, const rgg_box *__restrict__ old_b,
                                          const rgg_box *__restrict__ new_b, int32_t n_fixed)
{
    constexpr int kHalf = kDiffBlock / 2;
    __shared__ int s_tot[kDiffBlock / 64];
    __shared__ int s_bad, s_mism, s_base, s_any;
    const int tid = threadIdx.x, lane = lane_id(), wave = tid >> 6;
    const int side = tid / kHalf;        // 0: the old box's entry, 1: the new box's
    const int j = tid - side * kHalf;    // slot within the chunk
    if (tid == 0) {
        s_bad = 0;
        s_mism = 0;
        s_base = 0;
        s_any = 0;
        rm.ctl->n_items = 0;
        rm.ctl->claim = 0;
        rm.ctl->label_ticket = 0;
    }
    for (int t = tid; t < rm.ntiles; t += kDiffBlock) rm.tile_state[t] = 0ull;
    __syncthreads();
    bool dirty0 = false;   // the first chunk's slot changes (kept for the commit)
    rgg_box n0;
    for (int64_t base = 0; base < rm.M; base += kHalf) {
        const int64_t k = base + j;
        bool emit = false;
        rgg_box b;
        if (k < rm.M) {
            const rgg_box o = old_b[k], n = new_b[k], r = rm.resident[k];
            if (side == 0) {
                if (!box_ok(o) || !box_ok(n)) atomicOr(&s_bad, 1);
                if (!same_box(o, r)) atomicOr(&s_mism, 1);
            } else if (base == 0) {
                dirty0 = !same_box(n, r);
                n0 = n;
            }
            b = side ? n : o;
            emit = !same_box(o, n) && present<D>(b);
        }
        const uint64_t bm = __ballot(emit);
        if (lane == 0) s_tot[wave] = __popcll(bm);
        __syncthreads();
        int pos = s_base, tot = 0;
        for (int w = 0; w < kDiffBlock / 64; ++w) {
            if (w < wave) pos += s_tot[w];
            tot += s_tot[w];
        }
        pos += __popcll(bm & lanes_below());
        if (emit && write_entry<D>(rm, pos, b, side ? +1 : -1)) s_any = 1;
        __syncthreads();
        if (tid == 0) s_base += tot;
        __syncthreads();
    }
    const int status = s_bad ? RGG_E_INVALID_ARG : (s_mism ? RGG_E_STATE_MISMATCH : RGG_OK);
    if (tid == 0) {
        rm.ctl->status = status;
        rm.ctl->n_chg = status ? 0 : s_base;
        // fixed items are all looked at as soon as one changed box lies
        // inside the grid
        if (n_fixed) rm.ctl->n_items = (status == RGG_OK && s_any) ? n_fixed : 0;
    }
    if (status == RGG_OK) {
        if (dirty0) rm.resident[j] = n0;
        for (int64_t k = kHalf + tid; k < rm.M; k += kDiffBlock) {
            rgg_box n = new_b[k];
            if (!same_box(n, rm.resident[k])) rm.resident[k] = n;
        }
        // the entries written above are read back by this block's threads
        if (!n_fixed) {
            __syncthreads();
            activate_cells(rm, s_base);
        }
    }
}

template <int D>
__global__ void __launch_bounds__(kDiffBlock) k_diff(RmDev rm, const rgg_box *__restrict__ old_b,
                                                     const rgg_box *__restrict__ new_b)
{
    diff_body<D>(rm, old_b, new_b, rm.n_fixed);
}

// ------------------------------------------------------------------------
// block-level helpers
// ------------------------------------------------------------------------

// exclusive prefix of v over the block; *total receives the block sum.
// Contains barriers: every thread must call it.
template <int kNW = kWaves>
__device__ inline int block_scan(int v, int *total, int *wsum)
{
    const int lane = lane_id(), wv = threadIdx.x >> 6;
    int wt;
    const int pre = wave_prefix(v, &wt);
    __syncthreads();
    if (lane == 0) wsum[wv] = wt;
    __syncthreads();
    int off = 0, tot = 0;
    for (int w = 0; w < kNW; ++w) {
        off += w < wv ? wsum[w] : 0;
        tot += wsum[w];
    }
    *total = tot;
    return off + pre;
}

// Adds the counter deltas of one edge as fire-and-forget atomics (no value is
// returned, so they cost no round trip; integer adds commute, so the result
// does not depend on their order).
__device__ inline void add_counts(const RmDev &rm, int64_t e, int dC, int dS)
{
    int *c = reinterpret_cast<int *>(rm.cnt + e);
    if (dC) __hip_atomic_fetch_add(c, dC, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (dS) __hip_atomic_fetch_add(c + 1, dS, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

__device__ inline int32_t clamp_cell(double x, double org, double inv, int32_t n)
{
    int32_t c = cell_of(x, org, inv, n);
    return c < 0 ? 0 : (c > n - 1 ? n - 1 : c);
}

// ------------------------------------------------------------------------
// sphere samples: per edge a [B][J][S] block at S * soff[e], S values per copy
// (xyz + pad in 3-D, xy in 2-D), so one copy is one aligned vector load
// ------------------------------------------------------------------------

template <int D>
__host__ __device__ constexpr int copy_stride()
{
    return D == 3 ? kCopyStride3 : kCopyStride2;
}

// copy `idx` (= soff[e] + sphere * J + configuration) of the sample array
template <int D, typename T>
__device__ inline void load_copy(const T *samp, int64_t idx, T (&q)[D])
{
    const T *p = samp + copy_stride<D>() * idx;
    if constexpr (std::is_same<T, float>::value && D == 3) {
        const float4 v = *reinterpret_cast<const float4 *>(p);
        q[0] = v.x;
        q[1] = v.y;
        q[2] = v.z;
    } else if constexpr (std::is_same<T, float>::value && D == 2) {
        const float2 v = *reinterpret_cast<const float2 *>(p);
        q[0] = v.x;
        q[1] = v.y;
    } else {
#pragma unroll
        for (int k = 0; k < D; ++k) q[k] = p[k];
    }
}

// ------------------------------------------------------------------------
// binary64 re-test of an (edge, box) pair by one wavefront: the definition
// (C = some capsule meets, S = some sphere's capsule and one of its copies
// meet), used for the pairs whose binary32 decision fell inside the band
// ------------------------------------------------------------------------

struct CopyMap {
    int J, jw, spc, sub, jj;
};

__device__ inline CopyMap copy_map(int J)
{
    CopyMap c;
    c.J = J;
    c.jw = J < 64 ? J : 64;
    c.spc = 64 / c.jw;
    c.sub = lane_id() / c.jw;
    c.jj = lane_id() - c.sub * c.jw;
    return c;
}

template <int D>
__device__ bool copies_meet64(const RmDev &rm, const double *sb, const CopyMap &cm, uint64_t m,
                              const double *lo, const double *hi, const double *rad, int *lst,
                              unsigned long long *bytes)
{
    const int lane = lane_id();
    if (lane < rm.B && ((m >> lane) & 1ull)) lst[__popcll(m & lanes_below())] = lane;
    wave_sync();
    const int nsph = __popcll(m);
    // (spheres, configurations) in wavefront-sized pieces, two in flight
    const int nj = (cm.J + cm.jw - 1) / cm.jw, n = ((nsph + cm.spc - 1) / cm.spc) * nj;
    bool met = false;
    for (int k0 = 0; k0 < n && !met; k0 += 2) {
        double p[2][D], r[2];
        bool valid[2];
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            const int sp = ((k0 + u) / nj) * cm.spc + cm.sub, js = ((k0 + u) % nj) * cm.jw + cm.jj;
            valid[u] = k0 + u < n && cm.sub < cm.spc && sp < nsph && js < cm.J;
            r[u] = 0.0;
            if (valid[u]) {
                const int i = lst[sp];
#pragma unroll
                for (int k = 0; k < D; ++k) p[u][k] = sb[((int64_t)i * cm.J + js) * copy_stride<D>() + k];
                r[u] = rad[i];
            }
        }
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            const bool hit = valid[u] && point_box64<D>(p[u], lo, hi) <= r[u] * r[u];
            *bytes += (unsigned long long)(__popcll(__ballot(valid[u])) * D * 8);
            met = met || __ballot(hit);
        }
    }
    wave_sync();
    return met;
}

// some kept spline segment of a sphere in m meets the box (binary64, one
// wavefront: the spheres in turn, their segments across the lanes)
template <int D>
__device__ bool splines_meet64(const RmDev &rm, int64_t e, uint64_t m, const double *lo, const double *hi,
                               unsigned long long *bytes)
{
    constexpr int W = 2 * D + 1;
    const int lane = lane_id();
    while (m) {
        const int i = __ffsll((unsigned long long)m) - 1;
        m &= m - 1;
        const int64_t k = e * rm.B + i;
        const int32_t k0 = rm.sseg[k], k1 = rm.sseg[k + 1];
        for (int32_t j0 = k0; j0 < k1; j0 += 64) {
            const int32_t j = j0 + lane;
            bool hit = false;
            if (j < k1) {
                const double *g = rm.seg64 + (int64_t)j * W;
                double A[D], Bq[D];
#pragma unroll
                for (int d = 0; d < D; ++d) {
                    A[d] = g[d];
                    Bq[d] = g[D + d];
                }
                hit = segbox64<D>(A, Bq, lo, hi) <= g[2 * D] * g[2 * D];
            }
            *bytes += (unsigned long long)(min(64, k1 - j0) * W * 8);
            if (__ballot(hit)) return true;
        }
    }
    return false;
}

// ------------------------------------------------------------------------
// k_item: one block per work item (grid cell c, a chunk of at most 512 of
// its edges; the chunk size is the roadmap's work-item size).
//
//   1. every thread owns up to two edges of the item.  The changed entries
//      covering the cell are staged in LDS (tiles of kSubTile) and, when there
//      are many, registered in block-local slab masks; a thread ANDs the masks
//      of its edge's slabs and marks the candidates whose box meets its edge's
//      box, 32 per LDS word.  With several grid cells a pair is taken only by
//      the cell holding the lower corner of the two boxes' intersection, so
//      each (edge, entry) pair is tested once.
//      An item's start was five dependent rounds of loads (7 us of a block's
//      16 on small roadmaps); its loads are now requested together as far as
//      they do not depend on one another.
//   2. outer test, lanes = (pair, sphere): the capsule's ends are two of the
//      sphere's copies, and one that meets settles the pair (S is an existence
//      test, and S implies C); separation and end-sphere tests settle most of
//      the rest, and the tests left open are queued in LDS and run densely
//      with the exact segment-box minimum.
//   3. probe: a queued capsule that meets tests the copy nearest to where its
//      axis came closest to the box.
//   4. inner test of the pairs still open, rows = (pair, sphere whose capsule
//      met), lanes = configurations: every copy of those spheres.
//      The end copies settle most pairs that end RED before any exact test or
//      copy: an update of 290k spatial edges with 100 changed boxes 78.2 ->
//      75.0 us; in binary64, where every capsule ran the exact minimum (seven
//      divisions), 47.5 -> 37.1 us on 11.6k planar edges and 70.4 -> 53.3 on
//      46k spatial ones.
//   5. per pair C and S; the edge's counter deltas are summed in LDS and
//      added once per edge.  In FP32 a pair whose decision fell inside the
//      rounding band is queued and decided in binary64 by the same block
//      (retest_queued), after the item's rounds or when the queue fills.
// ------------------------------------------------------------------------

constexpr int kSubTile = 128;             // changed entries staged per tile
constexpr int kSlots = 2;                 // edge slots per thread
constexpr int kItemCap = kSlots * kBlock; // edges per work item at most
constexpr int kSlabMin = 33;              // staged entries from which the slab masks are made: an
                                          // edge tests one word's worth itself (spatial, 29k edges,
                                          // 12 changed boxes: 41.6 us with the masks, 39.8 without)
constexpr int kWords = kSubTile / 32;     // overlap words per edge
constexpr int kPairCap = kBlock;          // pairs per round (one per thread)
constexpr int kRowCap = 256;              // (pair, sphere) rows per copy round
constexpr int kOpenCap = 1024;            // capsule tests queued for the exact part
constexpr int kRetestCap = kPairCap + kRcCap;  // pairs queued for the binary64 re-test: what
                                          // may be waiting before a round, and the round
static_assert(kWords == 4, "a slab mask holds one uint4 of entry bits");
static_assert(kSubTile <= 65536 && kItemCap <= 65536, "a pair is (edge slot << 16) | entry in 32 bits");
static_assert(kLocalCells * 4 == kWords * kItemCap, "the overlap words reuse the slab masks' storage");
static_assert(2 * 3 * slabs_of(3) <= kLocalCells && 2 * 2 * slabs_of(2) <= kLocalCells && slabs_of(2) <= 128 &&
                  slabs_of(3) <= 128,
              "the slab masks fit their storage and one wavefront's scan (two slabs a lane)");
static_assert(kOpenCap >= 3 * kRowCap + 1, "the rows fit the capsule queue's storage");
static_assert(kOpenCap >= kWaves * 64, "the re-test's scratch fits the queue's storage");

__device__ inline int pe_slot(uint32_t v) { return (int)(v >> 16); }
__device__ inline int pe_entry(uint32_t v) { return (int)(v & 0xFFFFu); }

template <typename T>
struct ExactBoxes {
    T lo[3][kSubTile], hi[3][kSubTile];
};
struct NoBoxes {};
struct Radii32 {
    float r32[64];                        // sphere radii, binary32 (for the band)
};
struct NoRadii {};
struct RetestQueue {
    int2 pair[kRetestCap];
    int n;
};
struct NoQueue {};

template <typename T>
struct ItemLds {
    float4 blo[kSubTile], bhi[kSubTile];  // binary32 boxes: (lo, sbox), (hi, 0)
    int sign[kSubTile], gidx[kSubTile];
    // binary64 boxes for the binary64 kernel (the binary32 ones serve FP32)
    typename std::conditional<std::is_same<T, double>::value, ExactBoxes<double>, NoBoxes>::type x;
    typename std::conditional<std::is_same<T, float>::value, Radii32, NoRadii>::type r;
    union {
        // slab masks: sm[(2 d + 0) n + s] the staged entries whose slab range
        // on axis d starts at or before slab s, sm[(2 d + 1) n + s] those
        // whose range ends at or after it (n = slabs_of(D))
        uint4 sm[kLocalCells];
        uint32_t om[kWords][kItemCap];    // then the staged entries each edge's box meets
    } g;
    uint32_t cfg0[kItemCap];              // first configuration of each edge (sample / B)
    int edge[kItemCap], ej[kItemCap];     // edge id, configurations per sphere
    float es[kItemCap];                   // edge s (largest |coordinate| of its box)
    int dC[kItemCap], dS[kItemCap];
    uint32_t pe[kPairCap];                // edge slot << 16 | staged entry
    unsigned long long hm[kPairCap], um[kPairCap];
    // the capsule-test queue is dead once the exact part has run; the rows
    // and their copy offsets live after it, in the same storage, and between
    // rounds it is the scratch of the binary64 re-test
    union alignas(8) {
        uint32_t open[kOpenCap];          // queued (pair << 6 | sphere) capsule tests
        struct {
            uint32_t row[kRowCap];        // pair << 6 | sphere
            uint32_t rcopy[kRowCap + 1];
            uint32_t rbase[kRowCap];      // splines: the row's first segment
        } rw;
    } u;
    int nopen;
    uint32_t sf[kPairCap];
    int wsum[kWaves];
    // pairs (edge, changed entry) queued for the binary64 re-test
    typename std::conditional<std::is_same<T, float>::value, RetestQueue, NoQueue>::type r64;
    int pl_n;                             // pairs this block listed (pair listing)
    unsigned long long acc[kStats];
};

template <int D, typename T>
__device__ inline bool pair_owned(const RmDev &rm, const float4 &bl, const T *lo32, int64_t c)
{
    // lower corner of the intersection of the edge box and the entry box
    int64_t cell = 0, mul = 1;
    for (int k = 0; k < D; ++k) {
        const float ek = k == 0 ? bl.x : (k == 1 ? bl.y : bl.z);
        const float x = fmaxf(ek, (float)lo32[k]);
        cell += (int64_t)clamp_cell((double)x, rm.gorg[k], rm.ginv, rm.gdim[k]) * mul;
        mul *= rm.gdim[k];
    }
    return cell == c;
}

// Rounding band of a binary32 margin (squared-distance units): tau (s + R)
// (R + L) + tau^2 s^2, where s bounds every coordinate of the pair, R is the
// radius tested and L the L1 length of the capsule axis (0 for a sphere).
// The margin's rounding error is below 28 u s (R + L) + 7 u R^2 + O(u^2 s^2)
// (u = 2^-24), so tau = 1e-5 (about 168 u) leaves a factor of six.  The
// derivation assumes s <= 2^20 R; beyond that every decision is re-tested.
__device__ inline float band_of(float tau, float s, float R, float L)
{
    if (!(s <= 1048576.0f * R)) return INFINITY;
    return tau * (s + R) * (R + L) + (s > 0.0f ? tau * tau * s * s : 0.0f);
}

// Slab of coordinate x on axis d of the block-local slab masks, clamped to
// [0, n).  The subtraction, the product and floor are monotone, so the slab
// ranges of two boxes that share a point overlap on every axis.
__device__ inline int slab_of(const RmDev &rm, int d, float x, int n)
{
    const float f = floorf((x - rm.sl_org[d]) * rm.sl_inv[d]);
    return (int)fminf(fmaxf(f, 0.0f), (float)(n - 1));
}

// Binary64 counterpart of the band, for the quick tests of the binary64
// kernel: a decision farther than this from the threshold is what the binary64
// definition computes, whatever its rounding (every term of a squared distance
// is made of coordinates at most s + L in size and gaps; 1e-12 is about 9,000
// roundings of each).  As wide as the capsule test's also where an end copy is
// tested, so that a copy that meets implies its capsule does.
__device__ inline double band64_of(double s, double R, double L)
{
    if (!(s <= 1048576.0 * R)) return INFINITY;
    return 1e-12 * ((s + R) * (R + L) + L * L);
}

__device__ inline float max_of(float a, float b) { return fmaxf(a, b); }
__device__ inline double max_of(double a, double b) { return fmax(a, b); }
__device__ inline float min_of(float a, float b) { return fminf(a, b); }
__device__ inline double min_of(double a, double b) { return fmin(a, b); }
template <int D>
__device__ inline float point_box_of(const float *c, const float *lo, const float *hi)
{
    return point_box32<D>(c, lo, hi);
}
template <int D>
__device__ inline double point_box_of(const double *c, const double *lo, const double *hi)
{
    return point_box64<D>(c, lo, hi);
}

// Capsule i of edge e: its ends, radius and the L1 length of its axis.  The
// binary32 capsules are read as aligned 16-byte words, (A, R) and (B, L1) in
// 3-D, (A, B) and the radius beside it in 2-D: two loads from one address
// where the [2D + 1][B] rows of the binary64 ones took seven, each with an
// address of its own, in a phase that is bound by instruction issue.
template <int D>
__device__ __forceinline__ void load_capsule(const RmDev &rm, int e, int i, float (&A)[D], float (&Bq)[D], float &R,
                                             float &len)
{
    const int64_t k = (int64_t)e * rm.B + i;
    const float4 *q = reinterpret_cast<const float4 *>(rm.cap32);
    if constexpr (D == 3) {
        const float4 a = q[2 * k], b = q[2 * k + 1];
        A[0] = a.x;
        A[1] = a.y;
        A[2] = a.z;
        R = a.w;
        Bq[0] = b.x;
        Bq[1] = b.y;
        Bq[2] = b.z;
        len = b.w;
    } else {
        const float4 a = q[k];
        A[0] = a.x;
        A[1] = a.y;
        Bq[0] = a.z;
        Bq[1] = a.w;
        R = rm.capr32[k];
        len = fabsf(a.z - a.x) + fabsf(a.w - a.y);
    }
}

template <int D>
__device__ __forceinline__ void load_capsule(const RmDev &rm, int e, int i, double (&A)[D], double (&Bq)[D], double &R,
                                             double &len)
{
    const int B = rm.B;
    const double *cp = rm.cap64 + (int64_t)e * (2 * D + 1) * B;
    len = 0.0;
#pragma unroll
    for (int d = 0; d < D; ++d) {
        A[d] = cp[d * B + i];
        Bq[d] = cp[(D + d) * B + i];
        len += fabs(Bq[d] - A[d]);
    }
    R = cp[2 * D * B + i];
}

// The last of n rows whose first unit is at most c.
__device__ inline int row_of(const uint32_t *first, int n, uint32_t c)
{
    int lo = 0, hi = n - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (first[mid] <= c) lo = mid;
        else hi = mid - 1;
    }
    return lo;
}

// Binary64 decisions of the pairs queued in L.r64, by the whole block: C and S
// by their definition (capsules, the oriented boxes, then copies or spline
// segments), added to the edges' counters.  A wavefront takes up to 64 / B
// pairs at a time, the capsules of all of them on its lanes, then the copies
// pair by pair.  The queue ends empty; L.u serves as scratch.
// A block re-tests its own pairs (a spatial update queues about one per two
// blocks) at the end of its item: a chain of two loads and the exact minimum,
// 4 us at the end of some blocks.  A kernel of its own for all blocks' pairs
// cost 8 to 11 us of every update: the prefix of the blocks' counts, four
// dependent loads and a launch.
template <int D, int MODE, typename Lds>
__device__ __forceinline__ void retest_queued(const RmDev &rm, Lds &L, const int *s_lane, uint32_t &n_outer)
{
    const int tid = threadIdx.x, lane = lane_id(), wv = tid >> 6;
    const int B = rm.B, Gw = 64 / B;
    int *lst = reinterpret_cast<int *>(&L.u) + wv * 64;
    const int n = L.r64.n;
    unsigned long long bytes = 0;
    const uint64_t gm = (B == 64 ? 0ull : 1ull << B) - 1ull;
    const int per = min(Gw, (n + kWaves - 1) / kWaves);
    const int slot = s_lane[lane] >> 8, ci = s_lane[lane] & 255;
    for (int q0 = wv * per; q0 < n; q0 += kWaves * per) {
        const int m = min(per, n - q0);
        bool hit = false;
        if (slot < m) {
            const int2 pr = L.r64.pair[q0 + slot];
            const ChgEntry &en = rm.chg[pr.y];
            const double *cp = rm.cap64 + (int64_t)pr.x * (2 * D + 1) * B;
            double A[D], Bp[D], lo[D], hi[D];
#pragma unroll
            for (int d = 0; d < D; ++d) {
                A[d] = cp[d * B + ci];
                Bp[d] = cp[(D + d) * B + ci];
                lo[d] = en.lo[d];
                hi[d] = en.hi[d];
            }
            const double R = cp[2 * D * B + ci];
            hit = segbox64<D>(A, Bp, lo, hi) <= R * R;
        }
        const uint64_t hits = __ballot(hit);
        bytes += (unsigned long long)m * (2 * D + 1) * B * 8;
        for (int g = 0; g < m; ++g) {
            uint64_t hm = (hits >> (g * B)) & gm;
            if (!hm) continue;
            const int2 pr = L.r64.pair[q0 + g];
            const int64_t e = pr.x;
            const ChgEntry &en = rm.chg[pr.y];
            double lo[D], hi[D];
#pragma unroll
            for (int d = 0; d < D; ++d) {
                lo[d] = en.lo[d];
                hi[d] = en.hi[d];
            }
            if constexpr ((MODE & kModeObb) != 0) {
                // spheres whose body's oriented box misses are dropped
                bool keep = false;
                uint64_t sp = 0;
                if (lane < rm.nbody) {
                    sp = rm.body_sph[lane];
                    if (sp & hm) {
                        keep = obb_box_meet64<D>(rm.obb64 + (e * rm.nbody + lane) * obb_words(D), lo, hi);
                        bytes += lane == 0 ? obb_words(D) * 8 : 0;
                    }
                }
                uint64_t allowed = keep ? sp : 0ull;
                for (int o = 32; o > 0; o >>= 1) allowed |= __shfl_xor(allowed, o);
                hm &= allowed;
                if (!hm) continue;
            }
            bool S;
            if constexpr ((MODE & kModeSplines) != 0) {
                S = splines_meet64<D>(rm, e, hm, lo, hi, &bytes);
            } else {
                const int64_t s0 = rm.p_fixed ? e * rm.p_fixed : rm.soff[e];
                const int64_t P = rm.p_fixed ? rm.p_fixed : rm.soff[e + 1] - s0;
                const CopyMap cm = copy_map((int)(P / B));
                S = copies_meet64<D>(rm, rm.samp64 + copy_stride<D>() * s0, cm, hm, lo, hi, rm.rad64, lst, &bytes);
            }
            if (lane == 0) {
                ++n_outer;
                add_counts(rm, e, en.sign, S ? en.sign : 0);
            }
        }
    }
    if (lane == 0) atomicAdd(&L.acc[kStatFp64Bytes], bytes);
    __syncthreads();
    if (tid == 0) {
        L.acc[2] += (unsigned long long)n;
        L.r64.n = 0;
    }
    __syncthreads();
}

// One round of at most kPairCap pairs listed in L.pe (edge slot << 16 |
// entry): the outer test (capsules, then the oriented boxes), the probe, the
// inner test (copies or spline segments) and the decisions.  Item blocks
// (kShare false) sum each edge's counter deltas in L.dC / L.dS, pair-share
// blocks (kShare true: slot and entry are the pair itself) add the deltas to
// the counters at once.  Undecided pairs are queued in L.r64, which has room
// for a round (the caller re-tests them).
template <int D, typename T, int MODE, bool kShare, typename Lds>
__device__ __forceinline__ void test_round(const RmDev &rm, Lds &L, const T *s_rad2, const int *s_lane, int np,
                                           uint32_t &n_pairs, uint32_t &n_outer, unsigned long long &bytes)
{
    constexpr bool kF32 = std::is_same<T, float>::value;
    constexpr bool kObb = (MODE & kModeObb) != 0;
    constexpr bool kSpl = (MODE & kModeSplines) != 0;
    constexpr int kSegW = 2 * D + 1;   // values per spline segment
    const int tid = threadIdx.x, lane = lane_id(), wv = tid >> 6;
    const int B = rm.B;
    const int Gw = 64 / B;
    const T *samp = kF32 ? (const T *)rm.samp32 : (const T *)rm.samp64;
    const float band_rel = rm.band_rel;
    const int jfix = rm.p_fixed ? rm.p_fixed / B : 0;
    // coordinates of entry s in the kernel's precision
    auto box_lo = [&](int k, int s) -> T {
        if constexpr (kF32) return k == 0 ? L.blo[s].x : (k == 1 ? L.blo[s].y : L.blo[s].z);
        else return L.x.lo[k][s];
    };
    auto box_hi = [&](int k, int s) -> T {
        if constexpr (kF32) return k == 0 ? L.bhi[s].x : (k == 1 ? L.bhi[s].y : L.bhi[s].z);
        else return L.x.hi[k][s];
    };
    __syncthreads();   // the round's pairs are in L.pe
    n_pairs += np;
    // ---- outer test, quick part: lanes = (pair, sphere), the spheres of a
    // pair on consecutive lanes; each lane takes two pairs per step and issues
    // both capsules' loads first.  A capsule's ends are the sphere's first and
    // last copies, so an end within the sphere's own radius of the box settles
    // the whole pair (S, hence C): most pairs that end RED stop here, before
    // any exact test, probe or copy.  A separating axis is a certain miss, an
    // end within the capsule's radius a certain hit; what is left open is
    // queued for the exact part, which runs it on dense wavefronts.  "Certain"
    // is beyond the rounding band in both precisions.
    constexpr int kCapU = 2;
    const int slot = s_lane[lane] >> 8, ci = s_lane[lane] & 255;
    const uint64_t gm = (B == 64 ? 0ull : 1ull << B) - 1ull;   // a pair's lanes, from lane slot * B on
    for (int p0 = 0; p0 < np; p0 += kWaves * Gw * kCapU) {
        T A[kCapU][D], Bq[kCapU][D], R2[kCapU], L1[kCapU];
        int pu[kCapU];
#pragma unroll
        for (int u = 0; u < kCapU; ++u) {
            pu[u] = p0 + (u * kWaves + wv) * Gw + slot;
            R2[u] = T(0);
            L1[u] = T(0);
            if (slot < Gw && pu[u] < np)
                load_capsule<D>(rm, L.edge[pe_slot(L.pe[pu[u]])], ci, A[u], Bq[u], R2[u], L1[u]);
        }
#pragma unroll
        for (int u = 0; u < kCapU; ++u) {
            const int p = pu[u];
            const bool act = slot < Gw && p < np;
            int cls = kMiss;
            bool met = false;   // an end copy meets
            if (act) {
                const int s = pe_entry(L.pe[p]);
                T lo[D], hi[D];
#pragma unroll
                for (int k = 0; k < D; ++k) {
                    lo[k] = box_lo(k, s);
                    hi[k] = box_hi(k, s);
                }
                const float sc = fmaxf(L.es[pe_slot(L.pe[p])], L.blo[s].w);
                const T R = R2[u], RR = R * R;
                const T len = L1[u];
                T sep = T(0);
#pragma unroll
                for (int k = 0; k < D; ++k) {
                    sep = max_of(sep, max_of(lo[k] - max_of(A[u][k], Bq[u][k]), min_of(A[u][k], Bq[u][k]) - hi[k]));
                }
                T band, rband;
                if constexpr (kF32) {
                    band = band_of(band_rel, sc, R, len);
                    rband = band_of(band_rel, sc, L.r.r32[ci], 0.0f);
                } else {
                    band = band64_of((double)sc, R, len);
                    rband = band;
                }
                const T ends = min_of(point_box_of<D>(A[u], lo, hi), point_box_of<D>(Bq[u], lo, hi));
                met = !kSpl && ends - s_rad2[ci] < -rband;
                cls = (sep > T(0) && sep * sep - RR > band) ? kMiss : (ends - RR < -band ? kHit : kOpen);
            }
            const uint64_t metb = (__ballot(met) >> (slot * B)) & gm;
            const uint64_t hitb = (__ballot(cls == kHit) >> (slot * B)) & gm;
            if (act && ci == 0) {
                L.hm[p] = metb ? metb : hitb;
                L.um[p] = 0ull;
                L.sf[p] = metb ? 1u : 0u;
            }
            const bool op = act && cls == kOpen && !metb;
            const uint64_t ob = __ballot(op);
            if (ob) {
                int base = 0;
                if (lane == 0) base = atomicAdd(&L.nopen, __popcll(ob));
                base = __shfl(base, 0);
                if (op) {
                    const int q = base + __popcll(ob & lanes_below());
                    if (q < kOpenCap) {
                        L.u.open[q] = ((uint32_t)p << 6) | (uint32_t)ci;
                    } else if constexpr (kF32) {
                        atomicOr(&L.um[p], 1ull << ci);   // queue full: the binary64 re-test decides
                    } else {
                        const int s = pe_entry(L.pe[p]);   // queue full: decided at once
                        double lo[D], hi[D];
#pragma unroll
                        for (int k = 0; k < D; ++k) {
                            lo[k] = box_lo(k, s);
                            hi[k] = box_hi(k, s);
                        }
                        if (segbox64<D>(A[u], Bq[u], lo, hi) <= R2[u] * R2[u]) atomicOr(&L.hm[p], 1ull << ci);
                    }
                }
            }
        }
    }
    __syncthreads();
    {
        // ---- outer test, exact part: the queued tests, one per lane.  A
        // capsule that meets probes the copy nearest to where it came
        // closest: S is an existence test, so a copy found to meet settles the
        // pair.  In binary64 with the oriented boxes the sphere's box is not yet
        // known to meet, and there is no probe: the end copies settle most pairs
        // a probe would (with one behind the box test and none of them, an
        // update of 46k spatial edges took 68.3 us, now 46.4; of 56k arm edges 89.3
        // and 54.9; of 23k planar ones 47.0 and 28.7).
        constexpr bool kProbe = !kSpl && (kF32 || !kObb);
        const int nq = min(L.nopen, kOpenCap);
        for (int q = tid; q < nq; q += kBlock) {
            const uint32_t tk = L.u.open[q];
            const int p = (int)(tk >> 6), i = (int)(tk & 63u);
            const uint32_t pv = L.pe[p], te = pe_slot(pv), s = pe_entry(pv);
            T A[D], Bq[D], lo[D], hi[D], R, len;
            load_capsule<D>(rm, L.edge[te], i, A, Bq, R, len);
#pragma unroll
            for (int k = 0; k < D; ++k) {
                lo[k] = box_lo(k, s);
                hi[k] = box_hi(k, s);
            }
            const float sc = fmaxf(L.es[te], L.blo[s].w);
            int cls;
            float ts;
            if constexpr (kF32) {
                const float mg = segbox32<D>(A, Bq, lo, hi, ts) - R * R;
                cls = classify_margin(mg, band_of(band_rel, sc, R, len));
                if (cls == kUnsure) atomicOr(&L.um[p], 1ull << i);
            } else {
                double t64;
                cls = segbox64<D>(A, Bq, lo, hi, &t64) <= R * R ? kHit : kMiss;
                ts = (float)t64;
            }
            if (cls != kHit) continue;
            atomicOr(&L.hm[p], 1ull << i);
            if constexpr (kProbe) {
                if (__hip_atomic_load(&L.sf[p], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP)) continue;
                const int Je = L.ej[te];
                const int jj = min(Je - 1, (int)(fminf(fmaxf(ts, 0.0f), 1.0f) * (float)(Je - 1) + 0.5f));
                T c[D];
                load_copy<D>(samp, (int64_t)L.cfg0[te] * B + (int64_t)i * Je + jj, c);
                bytes += D * sizeof(T);
                bool meet;
                if constexpr (kF32)
                    meet = point_box32<D>(c, lo, hi) - s_rad2[i] < -band_of(band_rel, sc, L.r.r32[i], 0.0f);
                else
                    meet = point_box64<D>(c, lo, hi) <= s_rad2[i];
                if (meet) atomicOr(&L.sf[p], 1u);
            }
        }
        __syncthreads();
    }
    if constexpr (kObb) {
        // ---- oriented boxes: the outer part of sphere i is its
        // capsule intersected with its body's box, so a sphere
        // whose body's box misses is dropped (decided in binary64)
        if (tid < np) {
            const uint64_t cnd = L.hm[tid] | (kF32 ? L.um[tid] : 0ull);
            if (cnd && !L.sf[tid]) {
                const uint32_t pv = L.pe[tid], te = pe_slot(pv), s = pe_entry(pv);
                double lo[D], hi[D];
                if constexpr (kF32) {
                    const ChgEntry &en = rm.chg[L.gidx[s]];
#pragma unroll
                    for (int k = 0; k < D; ++k) {
                        lo[k] = en.lo[k];
                        hi[k] = en.hi[k];
                    }
                } else {
#pragma unroll
                    for (int k = 0; k < D; ++k) {
                        lo[k] = L.x.lo[k][s];
                        hi[k] = L.x.hi[k][s];
                    }
                }
                const double *ob = rm.obb64 + (int64_t)L.edge[te] * rm.nbody * obb_words(D);
                uint64_t keep = 0;
                for (int bd = 0; bd < rm.nbody; ++bd) {
                    const uint64_t sp = rm.body_sph[bd];
                    if (!(sp & cnd)) continue;
                    bytes += obb_words(D) * 8;
                    if (obb_box_meet64<D>(ob + bd * obb_words(D), lo, hi)) keep |= sp;
                }
                L.hm[tid] &= keep;
                if constexpr (kF32) L.um[tid] &= keep;
            }
        }
        __syncthreads();
    }
    // ---- rows: one per (open pair, sphere whose capsule met)
    const int p = tid;   // kPairCap == kBlock: this thread's pair
    uint64_t hmp = 0;
    int ra = 0;
    if (p < np) {
        hmp = L.hm[p];
        ra = L.sf[p] ? 0 : __popcll(hmp);
    }
    if (tid == 0) L.nopen = 0;   // for the next round
    int nrows;
    const int rpre = block_scan(ra, &nrows, L.wsum);
    __syncthreads();
    for (int q0 = 0; q0 < nrows; q0 += kRowCap) {
        const int nr = min(kRowCap, nrows - q0);
        if (ra > 0 && rpre < q0 + nr && rpre + ra > q0) {
            uint64_t m = hmp;
            int r = rpre;
            while (m && r < q0 + nr) {
                const int i = __ffsll((unsigned long long)m) - 1;
                m &= m - 1;
                if (r >= q0) L.u.rw.row[r - q0] = ((uint32_t)p << 6) | (uint32_t)i;
                ++r;
            }
        }
        __syncthreads();
        // the row's copies (spline segments): fixed count, or a scan
        // over the rows
        int ncopies = kSpl ? 0 : nr * jfix;
        if (kSpl || !jfix) {
            int cj[2], sum = 0;
            for (int h = 0; h < 2; ++h) {
                const int r = tid * 2 + h;
                cj[h] = 0;
                if (r < nr) {
                    const uint32_t rv = L.u.rw.row[r];
                    const int te = pe_slot(L.pe[rv >> 6]);
                    if constexpr (kSpl) {
                        const int64_t k = (int64_t)L.edge[te] * B + (int64_t)(rv & 63u);
                        const int32_t k0 = rm.sseg[k];
                        cj[h] = rm.sseg[k + 1] - k0;
                        L.u.rw.rbase[r] = (uint32_t)k0;
                    } else {
                        cj[h] = L.ej[te];
                    }
                }
                sum += cj[h];
            }
            const int cpre = block_scan(sum, &ncopies, L.wsum);
            int acc = cpre;
            for (int h = 0; h < 2; ++h) {
                const int r = tid * 2 + h;
                if (r < nr) L.u.rw.rcopy[r] = acc;
                acc += cj[h];
            }
            if (tid == 0) L.u.rw.rcopy[nr] = ncopies;
            __syncthreads();
        }
        // Each thread gathers kCopyU copies (all their loads in flight
        // together), then tests them.  Rows of more copies than one such pass
        // takes are clipped first: a copy lies within delta of the capsule
        // axis' point at its own parameter, so only the copies whose axis point
        // is within the capsule's radius of the box can meet it.  Their
        // parameters are an interval, inside the one where the axis is in the
        // box widened by that radius.  The clipped rows are dealt out in groups
        // of kCopyU consecutive copies, one group a thread at a time; a row
        // whose pair has already met the box is skipped.  (One pass is left
        // as it is: clipping costs a scan and a round of capsule loads.)
        // Planar edges hold up to a hundred copies per sphere: the binary64
        // update of 11.6k of them went from 37.1 to 32.6 us, a batch of 16
        // planar roadmaps from 75.4 to 71.9.
        constexpr int kCopyU = 4;
        const T *segb = kF32 ? (const T *)rm.seg32 : (const T *)rm.seg64;
        const bool clipped = !kSpl && ncopies > kBlock * kCopyU;
        int ngroups = 0;
        if (clipped) {
            int cnt = 0, first = 0;
            if (tid < nr) {
                const uint32_t rv = L.u.rw.row[tid];
                const int i = (int)(rv & 63u);
                const uint32_t pv = L.pe[rv >> 6], te = pe_slot(pv), s = pe_entry(pv);
                T A[D], Bq[D], R1, len;
                load_capsule<D>(rm, L.edge[te], i, A, Bq, R1, len);
                const float sc = fmaxf(L.es[te], L.blo[s].w), R = (float)R1;
                const float W = R + 1e-5f * (sc + R);   // far beyond rounding of any coordinate
                float t0 = 0.0f, t1 = 1.0f;
#pragma unroll
                for (int k = 0; k < D; ++k) {
                    const float A0 = (float)A[k], d = (float)(Bq[k] - A[k]);
                    const float a = (float)box_lo(k, s) - W - A0, b = (float)box_hi(k, s) + W - A0;
                    if (fabsf(d) > 1e-6f * (sc + R)) {   // else the axis stays inside what it is inside of
                        const float inv = __builtin_amdgcn_rcpf(d);
                        t0 = fmaxf(t0, fminf(a * inv, b * inv));
                        t1 = fminf(t1, fmaxf(a * inv, b * inv));
                    }
                }
                const int n = L.ej[te] - 1;
                const float slack = 0.01f + 1e-5f * (float)n;
                int last = n;
                if (t0 <= t1) {
                    first = max(0, (int)floorf(t0 * (float)n - slack));
                    last = min(n, (int)ceilf(t1 * (float)n + slack));
                }
                cnt = (last - first) / kCopyU + 1;
            }
            const int gpre = block_scan(cnt, &ngroups, L.wsum);
            __syncthreads();   // the rows' copy offsets are no longer read
            if (tid < nr) {
                L.u.rw.rcopy[tid] = (uint32_t)gpre;
                L.u.rw.rbase[tid] = (uint32_t)first;
            }
            __syncthreads();
        }
        const int nloop = clipped ? ngroups * kCopyU : ncopies;
        for (int c0 = 0; c0 < nloop; c0 += kBlock * kCopyU) {
            T q[kCopyU][kSpl ? kSegW : D];
            int cu_p[kCopyU], cu_i[kCopyU];
            int g_r = -1, g_j0 = 0;   // clipped: this thread's row and first copy index
            if (clipped) {
                const int f = c0 / kCopyU + tid;
                if (f < ngroups) {
                    g_r = row_of(L.u.rw.rcopy, nr, (uint32_t)f);
                    g_j0 = (int)(L.u.rw.rbase[g_r] + ((uint32_t)f - L.u.rw.rcopy[g_r]) * kCopyU);
                    // other waves may be setting the bit now: reading it
                    // late only costs a skipped skip
                    if (__hip_atomic_load(&L.sf[L.u.rw.row[g_r] >> 6], __ATOMIC_RELAXED,
                                          __HIP_MEMORY_SCOPE_WORKGROUP) & 1u)
                        g_r = -1;
                }
            }
            const int g_J = g_r >= 0 ? L.ej[pe_slot(L.pe[L.u.rw.row[g_r] >> 6])] : 0;
#pragma unroll
            for (int u = 0; u < kCopyU; ++u) {
                const int cidx = c0 + u * kBlock + tid;
                cu_p[u] = -1;
                cu_i[u] = 0;
                if (clipped ? g_j0 + u < g_J : cidx < ncopies) {
                    int r, jj;
                    if (clipped) {
                        r = g_r;
                        jj = g_j0 + u;
                    } else if (!kSpl && jfix) {
                        r = cidx / jfix;
                        jj = cidx - r * jfix;
                    } else {
                        r = row_of(L.u.rw.rcopy, nr, (uint32_t)cidx);
                        jj = cidx - (int)L.u.rw.rcopy[r];
                    }
                    const uint32_t rv = L.u.rw.row[r];
                    const int pp = (int)(rv >> 6);
                    const int i = (int)(rv & 63u);
                    const int te = pe_slot(L.pe[pp]);
                    if constexpr (kSpl) {
                        const T *sg = segb + ((int64_t)L.u.rw.rbase[r] + jj) * kSegW;
#pragma unroll
                        for (int k = 0; k < kSegW; ++k) q[u][k] = sg[k];
                    } else {
                        const int Je = L.ej[te];
                        load_copy<D>(samp, (int64_t)L.cfg0[te] * B + (int64_t)i * Je + jj, q[u]);
                    }
                    cu_p[u] = pp;
                    cu_i[u] = i;
                }
            }
#pragma unroll
            for (int u = 0; u < kCopyU; ++u) {
                const int pp = cu_p[u];
                if (pp < 0) continue;
                const uint32_t pv = L.pe[pp], te = pe_slot(pv), s = pe_entry(pv);
                T lo[D], hi[D];
#pragma unroll
                for (int k = 0; k < D; ++k) {
                    lo[k] = box_lo(k, s);
                    hi[k] = box_hi(k, s);
                }
                int cls;
                if constexpr (kSpl) {
                    // a spline segment: the capsule (A, B, rho)
                    T A[D], Bq[D];
#pragma unroll
                    for (int k = 0; k < D; ++k) {
                        A[k] = q[u][k];
                        Bq[k] = q[u][D + k];
                    }
                    const T rho = q[u][2 * D];
                    bytes += kSegW * sizeof(T);
                    if constexpr (kF32) {
                        const float sc = fmaxf(L.es[te], L.blo[s].w);
                        float len = 0.0f;
#pragma unroll
                        for (int k = 0; k < D; ++k) len += fabsf(Bq[k] - A[k]);
                        float ts;
                        const float mg = segbox32<D>(A, Bq, lo, hi, ts) - rho * rho;
                        cls = classify_margin(mg, band_of(band_rel, sc, rho, len));
                    } else {
                        cls = segbox64<D>(A, Bq, lo, hi) <= rho * rho ? kHit : kMiss;
                    }
                } else {
                    bytes += D * sizeof(T);
                    if constexpr (kF32) {
                        const float sc = fmaxf(L.es[te], L.blo[s].w);
                        cls = classify_margin(point_box32<D>(q[u], lo, hi) - s_rad2[cu_i[u]],
                                              band_of(band_rel, sc, L.r.r32[cu_i[u]], 0.0f));
                    } else {
                        cls = point_box64<D>(q[u], lo, hi) <= s_rad2[cu_i[u]] ? kHit : kMiss;
                    }
                }
                if (cls == kHit) atomicOr(&L.sf[pp], 1u);
                else if (cls == kUnsure) atomicOr(&L.sf[pp], 2u);
            }
        }
        __syncthreads();
    }
    // ---- decisions
    bool unsure = false;
    if (p < np) {
        const uint64_t ump = kF32 ? L.um[p] : 0ull;
        if (hmp || ump) {
            const uint32_t fp = L.sf[p];
            const uint32_t pv = L.pe[p], te = pe_slot(pv), s = pe_entry(pv);
            unsure = kF32 && (!hmp || (!(fp & 1u) && ((fp & 2u) || ump)));
            if (!unsure) {
                const int sign = L.sign[s];
                if constexpr (kShare) {
                    add_counts(rm, L.edge[te], sign, (fp & 1u) ? sign : 0);
                } else {
                    atomicAdd(&L.dC[te], sign);
                    if (fp & 1u) atomicAdd(&L.dS[te], sign);
                }
                ++n_outer;
            }
        }
    }
    if constexpr (kF32) {
        // undecided pairs are queued for the binary64 re-test
        const uint64_t ub = __ballot(unsure);
        if (ub) {
            int base = 0;
            if (lane == 0) base = atomicAdd(&L.r64.n, __popcll(ub));
            base = __shfl(base, 0);
            if (unsure) {
                const uint32_t pv = L.pe[p];
                L.r64.pair[base + __popcll(ub & lanes_below())] = make_int2(L.edge[pe_slot(pv)], L.gidx[pe_entry(pv)]);
            }
        }
    }
    __syncthreads();
}

// The block-local slab masks of the nt entries staged in L (masks zeroed
// before): each staged entry marks the slab its range starts in and the slab it
// ends in, on every axis; then each axis's start marks become "starts at or
// before s" (an OR over slabs 0..s) and its end marks "ends at or after s" (an
// OR over s..n-1): one wavefront per (axis, mark), each lane two slabs, the
// lanes joined by a wavefront scan.
template <int D, typename Lds>
__device__ __forceinline__ void slab_masks(const RmDev &rm, Lds &L, int nt)
{
    constexpr int kSl = slabs_of(D);
    const int tid = threadIdx.x, lane = lane_id(), wv = tid >> 6;
    if (tid < nt) {
        const float4 l = L.blo[tid], h = L.bhi[tid];
        const float lo3[3] = {l.x, l.y, l.z}, hi3[3] = {h.x, h.y, h.z};
        const uint32_t bit = 1u << (tid & 31);
        const int wd = tid >> 5;
        uint32_t *mw = reinterpret_cast<uint32_t *>(L.g.sm);
#pragma unroll
        for (int d = 0; d < D; ++d) {
            atomicOr(&mw[((2 * d) * kSl + slab_of(rm, d, lo3[d], kSl)) * 4 + wd], bit);
            atomicOr(&mw[((2 * d + 1) * kSl + slab_of(rm, d, hi3[d], kSl)) * 4 + wd], bit);
        }
    }
    __syncthreads();
    for (int a = wv; a < 2 * D; a += kWaves) {
        const bool up = (a & 1) == 0;   // start marks: forward
        uint4 *arr = L.g.sm + a * kSl;
        const int s0 = 2 * lane, s1 = 2 * lane + 1;
        auto at = [&](int s) -> uint4 & { return arr[up ? s : kSl - 1 - s]; };
        uint4 v0 = s0 < kSl ? at(s0) : make_uint4(0u, 0u, 0u, 0u);
        uint4 v1 = s1 < kSl ? at(s1) : make_uint4(0u, 0u, 0u, 0u);
        v1 = make_uint4(v1.x | v0.x, v1.y | v0.y, v1.z | v0.z, v1.w | v0.w);
        uint4 ex = v1;   // inclusive OR over lanes 0..lane, then shifted
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const uint32_t x = __shfl_up(ex.x, o), y = __shfl_up(ex.y, o), z = __shfl_up(ex.z, o),
                           w = __shfl_up(ex.w, o);
            if (lane >= o) ex = make_uint4(ex.x | x, ex.y | y, ex.z | z, ex.w | w);
        }
        uint4 pre = make_uint4(__shfl_up(ex.x, 1), __shfl_up(ex.y, 1), __shfl_up(ex.z, 1),
                               __shfl_up(ex.w, 1));
        if (lane == 0) pre = make_uint4(0u, 0u, 0u, 0u);
        if (s0 < kSl) at(s0) = make_uint4(pre.x | v0.x, pre.y | v0.y, pre.z | v0.z, pre.w | v0.w);
        if (s1 < kSl) at(s1) = make_uint4(pre.x | v1.x, pre.y | v1.y, pre.z | v1.z, pre.w | v1.w);
    }
}

// What staging takes of a changed entry, requested together.
struct Prefetched {
    float4 a, b;            // lo32[0..2], hi32[0]; hi32[1..2], sbox, sign
    int32_t c0[3], c1[3];
};

__device__ inline Prefetched fetch_entry(const ChgEntry &en)
{
    Prefetched p;
    const float4 *q = reinterpret_cast<const float4 *>(&en);
    p.a = q[0];
    p.b = q[1];
    for (int k = 0; k < 3; ++k) {
        p.c0[k] = en.c0[k];
        p.c1[k] = en.c1[k];
    }
    return p;
}

// Items li0, li0 + lstride, ... of the roadmap (statistics row blockIdx.x).
//
// The items are rm.fixed (fixed) or those that this update's cell activation
// emitted.  An item of the fixed list may lie in a cell that no changed box
// covers; it ends after its staging and counts for nothing.
//
// kList: the pair listing of the FP32 mode.  Each round of pairs goes to this
// block's region of the pair list (rm.pl, for the pair-share kernel) while
// the region has room; a round that does not fit is tested here, as the
// fused kernel does.
// kOne: item li0 alone, of an update that the caller knows to be valid.
template <int D, typename T, int MODE, bool kList = false, bool kOne = false>
__device__ __forceinline__ void item_body(const RmDev &rm, int li0, int lstride, bool fixed)
{
    constexpr bool kF32 = std::is_same<T, float>::value;
    static_assert(!kList || kF32, "the pair listing serves the FP32 mode");
    __shared__ ItemLds<T> L;
    __shared__ T s_rad2[64];
    const Ctl *ctl = rm.ctl;
    const int tid = threadIdx.x, lane = lane_id(), wv = tid >> 6;
    const int B = rm.B;
    // lane -> (pair slot, sphere) of the capsule phase, read from LDS where
    // needed rather than held in registers through the whole kernel
    __shared__ int s_lane[64];
    if (tid < 64) s_lane[tid] = ((tid / B) << 8) | (tid - (tid / B) * B);
    if (tid < kStats) L.acc[tid] = 0;
    if (tid < B) s_rad2[tid] = kF32 ? (T)rm.rad2_32[tid] : (T)(rm.rad64[tid] * rm.rad64[tid]);
    if constexpr (kF32) {
        if (tid < B) L.r.r32[tid] = (float)rm.rad64[tid];
    }
    if (tid == 0) {
        L.nopen = 0;
        if constexpr (kF32) L.r64.n = 0;
        L.pl_n = 0;
    }
    const bool single = rm.ncells == 1;
    const int4 *const items = fixed ? rm.fixed : rm.items;
    const int cap = kOne ? li0 + 1 : (single || fixed ? rm.n_fixed : (int)rm.items_cap);
    const int4 item0 = !single && li0 < cap ? items[li0] : make_int4(0, 0, 0, 0);
    const int status = kOne ? RGG_OK : ctl->status;
    // wavefront-uniform counts (kept in scalar registers) and per-lane ones
    uint32_t n_pairs = 0, visited = 0, cand = 0, n_outer = 0;
    unsigned long long bytes = 0;
    const int n_chg = ctl->n_chg;
    const int n_items = kOne ? cap : min(ctl->n_items, cap);
    const float4 *aabb = reinterpret_cast<const float4 *>(rm.aabb);
    const int jfix = rm.p_fixed ? rm.p_fixed / B : 0;
    constexpr int kSl = slabs_of(D);   // slabs per axis of the slab masks
    // where to go on: the item, its tile of changed entries, the tile's round
    // (not zero only after the re-test queue filled in the middle of an item)
    int it = li0, tile0 = 0, round0 = 0;
    bool full = true;
    uint32_t had = 0;   // bit h: edge slot h of the item has pairs
    while (full) {
        full = false;
        for (; it < cap && !full; it += full ? 0 : lstride) {
            const bool anew = tile0 == 0 && round0 == 0;
            // with one cell the items are chunks of the edges in order; else
            // slots of the cell lists.  What an item needs first is requested
            // in one go: the edges' slots and boxes and, beside them, the first
            // tile's entries (used when there are any), so that an item's
            // start waits for one round of loads with one cell and for three
            // (the item, the slots, the boxes) with several.
            int4 item = item0;
            if (single) item = make_int4(it * rm.chunk, (int)min((int64_t)rm.chunk, rm.E - (int64_t)it * rm.chunk), 0, 0);
            else if (it != li0) item = items[it];
            // (an emitted item is not looked at before it is known to be one)
            if (!single && !fixed && (status != RGG_OK || it >= n_items)) break;
            const int beg = item.x, n_e = item.y;   // edge slots in use: tid, tid + kBlock
            int e[kSlots], J[kSlots];
            float4 bl[kSlots], bh[kSlots];          // the edges' boxes: (lo, s), (hi, pad)
            uint32_t j0[kSlots];
#pragma unroll
            for (int h = 0; h < kSlots; ++h) {
                const int sl = tid + h * kBlock;
                e[h] = 0;
                J[h] = 0;
                j0[h] = 0;
                bl[h] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
                bh[h] = bl[h];
                if (sl < n_e) {
                    e[h] = beg + sl;
                    if (!single) {
                        // the cell list's slot: one contiguous load, no gather
                        const int4 cs = rm.cell_slot[beg + sl];
                        e[h] = cs.x;
                        j0[h] = (uint32_t)cs.y;
                        J[h] = cs.z;
                    } else if (jfix) {
                        J[h] = jfix;
                        j0[h] = (uint32_t)((int64_t)e[h] * jfix);
                    } else {
                        const int64_t s0 = rm.soff[e[h]];
                        j0[h] = (uint32_t)(s0 / B);
                        J[h] = (int)((rm.soff[e[h] + 1] - s0) / B);
                    }
                    bl[h] = aabb[2 * (int64_t)e[h]];
                    bh[h] = aabb[2 * (int64_t)e[h] + 1];
                }
            }
            Prefetched pf{};
            if (tid < kSubTile && tid < 2 * rm.M) pf = fetch_entry(rm.chg[tid]);
            // this block's place in the work, now that its loads are out
            if (status != RGG_OK || it >= n_items) break;
            const int c = item.z;
            const int cx = c % rm.gdim[0], cy = c / rm.gdim[0] % rm.gdim[1], cz = c / (rm.gdim[0] * rm.gdim[1]);
            __syncthreads();   // the previous item is done with the LDS arrays
#pragma unroll
            for (int h = 0; h < kSlots; ++h) {
                const int sl = tid + h * kBlock;
                L.edge[sl] = e[h];
                L.es[sl] = bl[h].w;
                L.cfg0[sl] = j0[h];
                L.ej[sl] = J[h];
                L.dC[sl] = 0;
                L.dS[sl] = 0;
            }
            if (tid == 0) {
                // every emitted item is visited once: clear the cell's mark
                // with its first chunk, so the next update starts from zero marks
                if (!single && !fixed && item.w == 0) atomicAnd(&rm.cell_bits[c >> 5], ~(1u << (c & 31)));
            }
            if (anew) had = 0;
            bool fused = !kList;   // some round of this item was tested here
            int n_round = 0;       // this item's pair rounds so far
            bool covered = kOne;   // some changed entry covers the item's cell
            if (kOne && anew) {
                if (wv == 0) visited += (uint32_t)n_e;
                bytes += (tid < n_e ? 32 : 0) + (tid + kBlock < n_e ? 32 : 0);
            }
            for (int j0 = tile0; j0 < n_chg && !full; j0 += kSubTile) {
                // stage the entries covering this cell (with one cell: all)
                const int j = j0 + tid;
                bool in = tid < kSubTile && j < n_chg;
                if (in) {
                    if (j0 > 0) pf = fetch_entry(rm.chg[j]);
                    in = single || (cx >= pf.c0[0] && cx <= pf.c1[0] && cy >= pf.c0[1] && cy <= pf.c1[1] &&
                                    cz >= pf.c0[2] && cz <= pf.c1[2]);
                }
                int nt = min(kSubTile, n_chg - j0), pos = tid;
                if (!single) pos = block_scan(in ? 1 : 0, &nt, L.wsum);
                if (in) {
                    L.blo[pos] = make_float4(pf.a.x, pf.a.y, pf.a.z, pf.b.z);
                    L.bhi[pos] = make_float4(pf.a.w, pf.b.x, pf.b.y, 0.0f);
                    L.sign[pos] = __float_as_int(pf.b.w);
                    if constexpr (!kF32) {
                        const ChgEntry &en = rm.chg[j];
                        for (int k = 0; k < 3; ++k) {
                            L.x.lo[k][pos] = en.lo[k];
                            L.x.hi[k][pos] = en.hi[k];
                        }
                    }
                    L.gidx[pos] = j;
                }
                pf = Prefetched{};   // not kept through the rounds
                if (nt == 0) continue;   // uniform: nt is the block total
                if constexpr (!kOne) {
                    if (anew && !covered) {
                        if (wv == 0) visited += (uint32_t)n_e;
                        bytes += (tid < n_e ? 32 : 0) + (tid + kBlock < n_e ? 32 : 0);
                    }
                    covered = true;
                }
                const int nw = (nt + 31) >> 5;
                // block-local slab masks, from kSlabMin entries on (below that
                // testing every entry costs less than the masks)
                const bool slabs = nt >= kSlabMin;
                if (slabs) {
                    for (int q = tid; q < 2 * D * kSl; q += kBlock) L.g.sm[q] = make_uint4(0u, 0u, 0u, 0u);
                    __syncthreads();
                    slab_masks<D>(rm, L, nt);
                }
                __syncthreads();
                // the staged entries each of this thread's edges meets, 32 per
                // word: the candidates whose slab range meets the edge's on
                // every axis (all reads of the slab masks first: their storage
                // then takes the words), then the exact test against the edge's
                // box
                uint32_t cw[kSlots][kWords];
                if (j0 != tile0) {   // a later tile: the boxes again
#pragma unroll
                    for (int h = 0; h < kSlots; ++h) {
                        const int sl = tid + h * kBlock;
                        if (sl < n_e) {
                            bl[h] = aabb[2 * (int64_t)L.edge[sl]];
                            bh[h] = aabb[2 * (int64_t)L.edge[sl] + 1];
                        }
                    }
                }
#pragma unroll
                for (int h = 0; h < kSlots; ++h) {
                    const int sl = tid + h * kBlock;
#pragma unroll
                    for (int w = 0; w < kWords; ++w) cw[h][w] = 0u;
                    if (sl < n_e) {
                        const float lo3[3] = {bl[h].x, bl[h].y, bl[h].z}, hi3[3] = {bh[h].x, bh[h].y, bh[h].z};
                        uint4 m = make_uint4(~0u, ~0u, ~0u, ~0u);
                        if (slabs) {
#pragma unroll
                            for (int d = 0; d < D; ++d) {
                                // entries starting at or before the edge's last
                                // slab and ending at or after its first
                                const uint4 st = L.g.sm[(2 * d) * kSl + slab_of(rm, d, hi3[d], kSl)];
                                const uint4 en = L.g.sm[(2 * d + 1) * kSl + slab_of(rm, d, lo3[d], kSl)];
                                m = make_uint4(m.x & st.x & en.x, m.y & st.y & en.y, m.z & st.z & en.z,
                                               m.w & st.w & en.w);
                            }
                        }
                        cw[h][0] = m.x;
                        cw[h][1] = m.y;
                        cw[h][2] = m.z;
                        cw[h][3] = m.w;
                    }
                }
                __syncthreads();
                int cnt = 0;
#pragma unroll
                for (int h = 0; h < kSlots; ++h) {
                    const int sl = tid + h * kBlock;
                    if (sl >= n_e) continue;
                    int ch = 0;
#pragma unroll
                    for (int w = 0; w < kWords; ++w) {
                        if (w < nw) {
                            const int left = nt - 32 * w;   // staged entries from this word on
                            uint32_t m = cw[h][w] & (left >= 32 ? ~0u : ((1u << left) - 1u)), bits = 0;
                            while (m) {
                                const int b = __ffs(m) - 1;
                                m &= m - 1;
                                const float4 l = L.blo[w * 32 + b], hb = L.bhi[w * 32 + b];
                                bool hit = (l.x <= bh[h].x) & (hb.x >= bl[h].x) & (l.y <= bh[h].y) & (hb.y >= bl[h].y) &
                                           (l.z <= bh[h].z) & (hb.z >= bl[h].z);
                                if (hit && !single) {
                                    const float lo3[3] = {l.x, l.y, l.z};
                                    hit = pair_owned<D, float>(rm, bl[h], lo3, c);
                                }
                                bits |= (uint32_t)hit << b;
                            }
                            L.g.om[w][sl] = bits;
                            ch += __popc(bits);
                        }
                    }
                    cnt += ch;
                    if (ch) had |= 1u << h;
                }
#pragma unroll
                for (int h = 0; h < kSlots; ++h) bl[h] = bh[h] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);   // not kept
                int tp;
                const int pre = block_scan(cnt, &tp, L.wsum);
                for (int r0 = j0 == tile0 ? round0 : 0; r0 < tp && !full; r0 += kPairCap) {
                    const int np = min(kPairCap, tp - r0);
                    if (cnt > 0 && pre < r0 + np && pre + cnt > r0) {
                        int k = pre;
                        for (int h = 0; h < kSlots && k < r0 + np; ++h) {
                            const int sl = tid + h * kBlock;
                            if (sl >= n_e) break;
                            for (int w = 0; w < nw && k < r0 + np; ++w) {
                                uint32_t m = L.g.om[w][sl];
                                while (m && k < r0 + np) {
                                    const int s = (w << 5) + __ffs(m) - 1;
                                    m &= m - 1;
                                    if (k >= r0) L.pe[k - r0] = ((uint32_t)sl << 16) | (uint32_t)s;
                                    ++k;
                                }
                            }
                        }
                    }
                    bool test = true;
                    if constexpr (kList) {
                        // after the item's first inline_rounds rounds, a round
                        // goes to the pair list when the region has room
                        if (n_round++ >= rm.inline_rounds) {
                            __syncthreads();   // the round's pairs are in L.pe
                            const int base = L.pl_n;
                            if (base + np <= rm.pl_cap) {
                                if (tid < np) {
                                    const uint32_t v = L.pe[tid];
                                    rm.pl[(int64_t)blockIdx.x * rm.pl_cap + base + tid] =
                                        make_int2(L.edge[pe_slot(v)], L.gidx[pe_entry(v)]);
                                }
                                bytes += tid < np ? 8 : 0;
                                __syncthreads();
                                if (tid == 0) L.pl_n = base + np;
                                __syncthreads();
                                test = false;
                            }
                        }
                        fused = fused || test;
                    }
                    if (test) test_round<D, T, MODE, false>(rm, L, s_rad2, s_lane, np, n_pairs, n_outer, bytes);
                    if constexpr (kF32) {
                        // no room for another round: re-test, then go on from here
                        if (L.r64.n >= rm.rc_cap) {
                            full = true;
                            tile0 = j0;
                            round0 = r0 + kPairCap;
                        }
                    }
                }
            }
            if (!full) tile0 = round0 = 0;
            if (!covered) continue;
            if (!full) cand += (uint32_t)(__popcll(__ballot(had & 1u)) + __popcll(__ballot(had & 2u)));
            if (fused && !full) bytes += (unsigned long long)__popc(had) * ((2 * D + 1) * B * sizeof(T) + 16);
            __syncthreads();
#pragma unroll
            for (int h = 0; h < kSlots; ++h) {
                const int sl = tid + h * kBlock;
                if (sl < n_e) add_counts(rm, L.edge[sl], L.dC[sl], L.dS[sl]);
            }
        }
        if constexpr (kF32) {
            __syncthreads();
            if (L.r64.n) retest_queued<D, MODE>(rm, L, s_lane, n_outer);
        }
    }
    __syncthreads();
    // per-lane counts are summed over the wavefront first: LDS atomics on
    // one address from every lane are slow
    const unsigned long long w_outer = wave_sum_u64(n_outer), w_bytes = wave_sum_u64(bytes);
    if (tid == 0 && n_pairs) atomicAdd(&L.acc[0], (unsigned long long)n_pairs);
    const int byte_row = kF32 && !kOne ? kStatItemBytes : kStatPairBytes;
    if (lane == 0) {
        if (w_outer) atomicAdd(&L.acc[1], w_outer);
        if (w_bytes) atomicAdd(&L.acc[byte_row], w_bytes);
        if (visited) atomicAdd(&L.acc[4], (unsigned long long)visited);
        if (cand) atomicAdd(&L.acc[5], (unsigned long long)cand);
    }
    __syncthreads();
    // statistic k at bs[k * kStatBlocks]: item blocks add to row blockIdx &
    // (kStatRows - 1), shared with other blocks (atomics)
    unsigned long long *bs = rm.blk_stats + (int)(blockIdx.x & (kStatRows - 1));
    if (tid < kStats && L.acc[tid]) atomicAdd(&bs[tid * kStatBlocks], L.acc[tid]);
    if (kList && tid == 0) rm.pl_cnt[blockIdx.x] = L.pl_n;
}

// The binary32 kernel is held to the registers with which kPerCu blocks fit on
// a CU (four: 128 VGPRs); the binary64 one keeps the compiler's choice.  An
// update that lists no pairs runs without the listing (kList false): on three
// roadmaps and obstacle walks each, 63.4 -> 62.5, 47.6 -> 47.0 and 32.1 -> 31.6
// us for the arm's second forms (93k edges), 64.0 -> 63.4, 58.0 -> 57.4 and 58.8 ->
// 58.1 for 290k spatial edges; planar edges and 464k arm edges take the same
// (28.3, 75.1 -> 75.4).
template <int D, int MODE, bool kList, int kPerCu>
__global__ void __launch_bounds__(kBlock, kPerCu) k_item32(RmDev rm)
{
    item_body<D, float, MODE, kList>(rm, (int)blockIdx.x, (int)gridDim.x, rm.n_fixed > 0);
}

template <int D, int MODE>
__global__ void __launch_bounds__(kBlock) k_item64(RmDev rm)
{
    item_body<D, double, MODE>(rm, (int)blockIdx.x, (int)gridDim.x, rm.n_fixed > 0);
}

// ------------------------------------------------------------------------
// k_pairs: the balanced pair testing of the FP32 mode (launched only when
// the item kernel lists pairs).  The listing leaves each block's pairs in
// its region of rm.pl; this kernel cuts the concatenation of the regions
// into equal shares, as many as the device holds at once while a share fits
// one round, so every block tests the same number of pairs whatever the
// items' sizes were.  A share runs in rounds of kPairCap pairs through the
// same phases as an item block's round (each pair is its own edge slot and
// entry); counter deltas go to the counters at once.
// ------------------------------------------------------------------------

struct ShareLds {
    float4 blo[kPairCap], bhi[kPairCap];  // the pairs' entries: (lo, sbox), (hi, 0)
    int sign[kPairCap], gidx[kPairCap];
    NoBoxes x;
    Radii32 r;
    uint32_t cfg0[kPairCap];              // first configuration of each pair's edge
    int edge[kPairCap], ej[kPairCap];     // edge id, configurations per sphere
    float es[kPairCap];                   // edge s (largest |coordinate| of its box)
    uint32_t pe[kPairCap];                // pair << 16 | pair
    unsigned long long hm[kPairCap], um[kPairCap];
    union alignas(8) {
        uint32_t open[kOpenCap];
        struct {
            uint32_t row[kRowCap];
            uint32_t rcopy[kRowCap + 1];
            uint32_t rbase[kRowCap];
        } rw;
    } u;
    int nopen;
    uint32_t sf[kPairCap];
    int wsum[kWaves];
    RetestQueue r64;
    int pref[kStatBlocks + 1];            // listed pairs before each region
    unsigned long long acc[kStats];
};

template <int D, int MODE>
__device__ __forceinline__ void share_body(const RmDev &rm)
{
    __shared__ ShareLds L;
    __shared__ float s_rad2[64];
    __shared__ int s_lane[64];
    const int tid = threadIdx.x, lane = lane_id();
    const int B = rm.B;
    if (tid < 64) s_lane[tid] = ((tid / B) << 8) | (tid - (tid / B) * B);
    if (tid < kStats) L.acc[tid] = 0;
    if (tid < B) {
        s_rad2[tid] = rm.rad2_32[tid];
        L.r.r32[tid] = (float)rm.rad64[tid];
    }
    if (tid == 0) {
        L.nopen = 0;
        L.r64.n = 0;
    }
    // prefix of the regions' pair counts: kPer consecutive regions per thread
    constexpr int kPer = kStatBlocks / kBlock;
    static_assert(kStatBlocks % kBlock == 0, "regions are scanned kPer per thread");
    int c[kPer], sum = 0;
#pragma unroll
    for (int k = 0; k < kPer; ++k) {
        c[k] = rm.pl_cnt[tid * kPer + k];
        sum += c[k];
    }
    int total;
    int pre = block_scan(sum, &total, L.wsum);
#pragma unroll
    for (int k = 0; k < kPer; ++k) {
        L.pref[tid * kPer + k] = pre;
        pre += c[k];
    }
    if (tid == 0) L.pref[kStatBlocks] = total;
    __syncthreads();
    // the shares: as many as fit on the device at once while each is at most
    // one round, more (up to the grid) when the pairs need more rounds; a
    // share then holds at most max(kPairCap, pl_cap) pairs
    const int G = min((int)gridDim.x, max(rm.test_slots, (total + kPairCap - 1) / kPairCap));
    const int b = (int)blockIdx.x;
    const int64_t lo = b < G ? (int64_t)total * b / G : 0;
    const int64_t hi = b < G ? (int64_t)total * (b + 1) / G : 0;
    const float4 *aabb = reinterpret_cast<const float4 *>(rm.aabb);
    const int jfix = rm.p_fixed ? rm.p_fixed / B : 0;
    uint32_t n_pairs = 0, n_outer = 0;
    unsigned long long bytes = 0;
    for (int64_t r0 = lo; r0 < hi; r0 += kPairCap) {
        const int np = (int)min((int64_t)kPairCap, hi - r0);
        if (tid < np) {
            // the pair's region: the last one whose first pair is at most g
            const int g = (int)(r0 + tid);
            int a = 0, z = kStatBlocks - 1;
            while (a < z) {
                const int m = (a + z + 1) >> 1;
                if (L.pref[m] <= g) a = m;
                else z = m - 1;
            }
            const int2 pr = rm.pl[(int64_t)a * rm.pl_cap + (g - L.pref[a])];
            const int e = pr.x, j = pr.y;
            const float4 *q = reinterpret_cast<const float4 *>(&rm.chg[j]);
            const float4 qa = q[0], qb = q[1];   // lo32[0..2], hi32[0]; hi32[1..2], sbox, sign
            L.blo[tid] = make_float4(qa.x, qa.y, qa.z, qb.z);
            L.bhi[tid] = make_float4(qa.w, qb.x, qb.y, 0.0f);
            L.sign[tid] = __float_as_int(qb.w);
            L.gidx[tid] = j;
            L.edge[tid] = e;
            L.es[tid] = aabb[2 * (int64_t)e].w;
            if (jfix) {
                L.ej[tid] = jfix;
                L.cfg0[tid] = (uint32_t)((int64_t)e * jfix);
            } else {
                const int64_t s0 = rm.soff[e];
                L.cfg0[tid] = (uint32_t)(s0 / B);
                L.ej[tid] = (int)((rm.soff[e + 1] - s0) / B);
            }
            L.pe[tid] = ((uint32_t)tid << 16) | (uint32_t)tid;
            // the pair record and entry, the edge's box word; its capsules
            // once per run of pairs of one edge
            bytes += 8 + 32 + 4;
        }
        __syncthreads();
        if (tid < np && (tid == 0 || L.edge[tid] != L.edge[tid - 1]))
            bytes += (unsigned long long)((2 * D + 1) * B * sizeof(float) + (jfix ? 0 : 16));
        test_round<D, float, MODE, true>(rm, L, s_rad2, s_lane, np, n_pairs, n_outer, bytes);
        if (L.r64.n) retest_queued<D, MODE>(rm, L, s_lane, n_outer);
    }
    __syncthreads();
    const unsigned long long w_outer = wave_sum_u64(n_outer), w_bytes = wave_sum_u64(bytes);
    if (tid == 0 && n_pairs) atomicAdd(&L.acc[0], (unsigned long long)n_pairs);
    if (lane == 0) {
        if (w_outer) atomicAdd(&L.acc[1], w_outer);
        if (w_bytes) atomicAdd(&L.acc[kStatPairBytes], w_bytes);
    }
    __syncthreads();
    // the statistics rows are shared by blocks (atomics)
    unsigned long long *bs = rm.blk_stats + (blockIdx.x & (kStatRows - 1));
    if (tid == 0) {
        if (L.acc[0]) atomicAdd(&bs[0], L.acc[0]);
        if (L.acc[1]) atomicAdd(&bs[1 * kStatBlocks], L.acc[1]);
        if (L.acc[2]) atomicAdd(&bs[2 * kStatBlocks], L.acc[2]);
        if (L.acc[kStatFp64Bytes]) atomicAdd(&bs[kStatFp64Bytes * kStatBlocks], L.acc[kStatFp64Bytes]);
        if (L.acc[kStatPairBytes]) atomicAdd(&bs[kStatPairBytes * kStatBlocks], L.acc[kStatPairBytes]);
    }
}

template <int D, int MODE>
__global__ void __launch_bounds__(kBlock, 4) k_pairs(RmDev rm)
{
    share_body<D, MODE>(rm);
}

// ------------------------------------------------------------------------
// labels and the ordered gray list
// ------------------------------------------------------------------------

__device__ inline uint8_t label_of(int2 c)
{
    return c.y > 0 ? (uint8_t)RGG_RED : (c.x == 0 ? (uint8_t)RGG_GREEN : (uint8_t)RGG_GRAY);
}

__device__ inline int block_sum(int v, int *s_w)
{
    for (int o = 32; o > 0; o >>= 1) v += __shfl_down(v, o);
    const int lane = lane_id(), wv = threadIdx.x >> 6;
    __syncthreads();
    if (lane == 0) s_w[wv] = v;
    __syncthreads();
    int t = 0;
    for (int w = 0; w < kWaves; ++w) t += s_w[w];
    return t;
}

// Each thread of a label block owns R consecutive edges of the tile: 16 in a
// block of 256 threads, 4 in one of 1,024.
constexpr int kLabelRun = kLabelTile / kBlock;
constexpr int kWideRun = 4;

template <int R>
__device__ inline void load_run(const RmDev &rm, int64_t e0, int2 (&c)[R])
{
    if (e0 + R <= rm.E) {
        const int4 *src = reinterpret_cast<const int4 *>(rm.cnt + e0);   // 16-byte aligned: e0 % R == 0
#pragma unroll
        for (int h = 0; h < R / 2; ++h) {
            const int4 v = src[h];
            c[2 * h] = make_int2(v.x, v.y);
            c[2 * h + 1] = make_int2(v.z, v.w);
        }
    } else {
#pragma unroll
        for (int h = 0; h < R; ++h) c[h] = e0 + h < rm.E ? rm.cnt[e0 + h] : make_int2(0, 0);
    }
}

// k_count: gray edges per tile
__device__ __forceinline__ void count_body(const RmDev &rm, int tile)
{
    __shared__ int s_w[kWaves];
    const int tid = threadIdx.x;
    const int64_t e0 = (int64_t)tile * kLabelTile + (int64_t)tid * kLabelRun;
    int2 c[kLabelRun];
    load_run(rm, e0, c);
    int ng = 0;
#pragma unroll
    for (int h = 0; h < kLabelRun; ++h) ng += (e0 + h < rm.E && label_of(c[h]) == RGG_GRAY) ? 1 : 0;
    const int tot = block_sum(ng, s_w);
    if (tid == 0) rm.tile_cnt[tile] = tot;
}

// Folds the statistics rows of the update into *res (when res is not null)
// and clears them for the next update (the item kernels add to them).
__device__ __forceinline__ void fold_stats(const RmDev &rm, rgg_update_result *res)
{
    __shared__ unsigned long long s_part[kWaves][kStats];
    const int tid = threadIdx.x;
    static_assert(kStatRows == kBlock, "one statistics row a thread");
    const bool on = tid < kStatRows;
    unsigned long long v[kStats];
#pragma unroll
    for (int k = 0; k < kStats; ++k) v[k] = on ? rm.blk_stats[k * kStatBlocks + tid] : 0ull;
#pragma unroll
    for (int k = 0; k < kStats; ++k)
        if (on) rm.blk_stats[k * kStatBlocks + tid] = 0ull;
    const int lane = lane_id(), wv = tid >> 6;
#pragma unroll
    for (int k = 0; k < kStats; ++k) {
        const unsigned long long w = wave_sum_u64(v[k]);
        if (on && lane == 0) s_part[wv][k] = w;
    }
    __syncthreads();
    if (tid == 0 && res) {
        int64_t a[kStats];
        for (int k = 0; k < kStats; ++k) {
            unsigned long long t = 0;
            for (int w = 0; w < kWaves; ++w) t += s_part[w][k];
            a[k] = (int64_t)t;
        }
        res->n_pairs = a[0];
        res->n_outer_hits = a[1];
        res->n_rechecked = a[2];
        res->test_bytes = a[kStatPairBytes] + a[kStatItemBytes] + a[kStatFp64Bytes];
        res->n_cells_visited = a[4];
        res->n_candidate_edges = a[5];
        res->item_bytes = a[kStatItemBytes];
        res->fp64_bytes = a[kStatFp64Bytes];
    }
}

// Labels of this thread's run of edges e0 .. e0 + R - 1; returns
// how many are GRAY.
template <int R>
__device__ __forceinline__ int run_labels(const RmDev &rm, int64_t e0, uint8_t (&lab)[R])
{
    int2 c[R];
    load_run(rm, e0, c);
    int ng = 0;
#pragma unroll
    for (int h = 0; h < R; ++h) {
        lab[h] = label_of(c[h]);
        ng += (e0 + h < rm.E && lab[h] == RGG_GRAY) ? 1 : 0;
    }
    return ng;
}

// Stores a run's labels (when labels is not null).
template <int R>
__device__ __forceinline__ void store_run(const RmDev &rm, uint8_t *labels, int64_t e0, const uint8_t (&lab)[R])
{
    if (!labels) return;
    static_assert(R == 16 || R == 4, "a run is stored as one label word");
    if (e0 + R <= rm.E && ((uintptr_t)(labels + e0) & (R - 1u)) == 0) {
        uint32_t wds[R / 4];
#pragma unroll
        for (int q = 0; q < R / 4; ++q)
            wds[q] = (uint32_t)lab[4 * q] | ((uint32_t)lab[4 * q + 1] << 8) | ((uint32_t)lab[4 * q + 2] << 16) |
                     ((uint32_t)lab[4 * q + 3] << 24);
        if constexpr (R == 16) *reinterpret_cast<uint4 *>(labels + e0) = make_uint4(wds[0], wds[1], wds[2], wds[3]);
        else *reinterpret_cast<uint32_t *>(labels + e0) = wds[0];
    } else {
#pragma unroll
        for (int h = 0; h < R; ++h)
            if (e0 + h < rm.E) labels[e0 + h] = lab[h];
    }
}

// Stores a tile's GRAY ids in ascending order from gray-list position
// `before` on (when gray is not null; ids past cap are dropped).  Each
// thread puts its run's ids in LDS at the tile-local positions pre, pre + 1,
// ..., then consecutive threads write consecutive positions, so the 8-byte
// stores coalesce instead of each thread's landing a few positions apart.
// Every thread of the block calls it (one barrier).
template <int R>
__device__ __forceinline__ void store_gray(const RmDev &rm, int64_t *gray, int64_t cap, int64_t e0,
                                           const uint8_t (&lab)[R], int64_t before, int pre, int tot)
{
    __shared__ uint16_t s_gid[kLabelTile];   // tile-local edge index of each GRAY id
    static_assert(kLabelTile <= 65536, "a tile-local index fits 16 bits");
    if (!gray) return;
    const int64_t t0 = e0 - (int64_t)threadIdx.x * R;   // the tile's first edge
    int p = pre;
#pragma unroll
    for (int h = 0; h < R; ++h)
        if (e0 + h < rm.E && lab[h] == RGG_GRAY) s_gid[p++] = (uint16_t)(threadIdx.x * R + h);
    __syncthreads();
    for (int i = threadIdx.x; i < tot; i += kLabelTile / R) {
        const int64_t pos = before + i;
        if (pos < cap) gray[pos] = t0 + s_gid[i];
    }
}

// k_write: labels and the ordered gray list, one tile per block (its first
// position is the sum of the earlier tiles' counts from k_count; the last
// tile reports n_gray, tile 0 the status); block `ntiles` instead folds the
// per-block statistics of the update.
__device__ __forceinline__ void write_body(const RmDev &rm, uint8_t *labels, int64_t *gray, int64_t cap,
                                          rgg_update_result *res, int force, int tile)
{
    __shared__ int s_w[kWaves];
    const int tid = threadIdx.x;
    if (tile == rm.ntiles) {
        if (!force) fold_stats(rm, res);
        return;
    }
    const int status = force ? RGG_OK : rm.ctl->status;
    if (tid == 0 && tile == 0 && res && !force) {
        res->status = status;
        res->n_changed = rm.ctl->n_chg;
        if (status != RGG_OK) res->n_gray = 0;
    }
    if (status != RGG_OK) return;
    const int64_t e0 = (int64_t)tile * kLabelTile + (int64_t)tid * kLabelRun;
    uint8_t lab[kLabelRun];
    const int ng = run_labels(rm, e0, lab);
    // gray edges before this tile
    int before = 0;
    for (int t = tid; t < tile; t += kBlock) before += rm.tile_cnt[t];
    before = block_sum(before, s_w);
    int tot;
    const int pre = block_scan(ng, &tot, s_w);
    if (tid == 0 && tile == rm.ntiles - 1 && res) res->n_gray = (int64_t)before + tot;
    if (tot == 0 && labels == nullptr) return;
    store_run(rm, labels, e0, lab);
    store_gray(rm, gray, cap, e0, lab, before, pre, tot);
}

// k_labels: k_count and k_write in one pass.  Blocks take their tiles in
// dispatch order (a ticket), publish their gray count, and add up the
// earlier tiles' counts by looking back over their published words,
// sixty-four at a time, stopping at the nearest tile that already published
// its inclusive prefix (the decoupled look-back scan of Merrill and Garland,
// "Single-pass Parallel Prefix Scan with Decoupled Look-back", 2016).  A
// block only waits on tiles whose blocks took earlier tickets and are
// therefore running, so every wait ends; the waits are bounded all the same
// and report RGG_E_DEVICE if a bound is ever reached.  The block with the
// last ticket folds the statistics.  k_diff clears the words and the ticket
// before each update.
constexpr unsigned long long kTileAgg = 1ull << 62, kTilePre = 2ull << 62, kTileVal = (1ull << 62) - 1;
constexpr int kLookBackSpins = 1 << 20;

template <int R>
__device__ __forceinline__ void labels_body(const RmDev &rm, uint8_t *labels, int64_t *gray, int64_t cap,
                                           rgg_update_result *res)
{
    constexpr int kThreads = kLabelTile / R;
    __shared__ int s_w[kThreads / 64];
    __shared__ int s_tile, s_fail;
    __shared__ long long s_before;
    const int tid = threadIdx.x, lane = lane_id(), wv = tid >> 6;
    if (tid == 0) s_tile = __hip_atomic_fetch_add(&rm.ctl->label_ticket, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __syncthreads();
    const int tile = s_tile;
    if (tile >= rm.ntiles) {
        // every block has its ticket: the counter starts from zero next time
        if (tid == 0) __hip_atomic_store(&rm.ctl->label_ticket, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        fold_stats(rm, res);
        return;
    }
    const int status = rm.ctl->status;
    if (tid == 0 && tile == 0 && res) {
        res->status = status;
        res->n_changed = rm.ctl->n_chg;
        if (status != RGG_OK) res->n_gray = 0;
    }
    if (status != RGG_OK) return;   // every block returns here: no one waits
    const int64_t e0 = (int64_t)tile * kLabelTile + (int64_t)tid * R;
    uint8_t lab[R];
    const int ng = run_labels(rm, e0, lab);
    int tot;
    const int pre = block_scan<kThreads / 64>(ng, &tot, s_w);
    unsigned long long *st = rm.tile_state;
    if (tid == 0)
        __hip_atomic_store(&st[tile], (tile == 0 ? kTilePre : kTileAgg) | (unsigned long long)tot, __ATOMIC_RELEASE,
                           __HIP_MEMORY_SCOPE_AGENT);
    if (wv == 0) {
        unsigned long long before = 0;
        bool fail = false;
        for (int t = tile - 1; t >= 0; t -= 64) {
            const int q = t - lane;              // lane l looks at tile t - l
            unsigned long long v = kTilePre;     // before tile 0: an inclusive prefix of 0
            bool ready = q < 0;
            for (int spin = 0;; ++spin) {
                if (!ready) {
                    v = __hip_atomic_load(&st[q], __ATOMIC_ACQUIRE, __HIP_MEMORY_SCOPE_AGENT);
                    ready = (v >> 62) != 0;
                }
                if (__ballot(!ready) == 0) break;
                if (spin >= kLookBackSpins) {
                    fail = true;
                    break;
                }
                __builtin_amdgcn_s_sleep(1);
            }
            if (fail) break;
            const uint64_t pm = __ballot((v >> 62) == 2);
            const int stop = pm ? __ffsll((unsigned long long)pm) - 1 : 63;
            before += wave_sum_u64(lane <= stop ? (v & kTileVal) : 0ull);
            if (pm) break;
        }
        if (lane == 0) {
            s_before = (long long)before;
            s_fail = fail ? 1 : 0;
        }
    }
    __syncthreads();
    const long long before = s_before;
    if (tid == 0) {
        __hip_atomic_store(&st[tile], kTilePre | (unsigned long long)(before + tot), __ATOMIC_RELEASE,
                           __HIP_MEMORY_SCOPE_AGENT);
        if (res && s_fail) res->status = RGG_E_DEVICE;
        if (res && tile == rm.ntiles - 1) res->n_gray = before + tot;
    }
    store_run(rm, labels, e0, lab);
    store_gray(rm, gray, cap, e0, lab, before, pre, tot);
}

template <int R>
__global__ void __launch_bounds__(kLabelTile / R) k_labels(RmDev rm, uint8_t *labels, int64_t *gray, int64_t cap,
                                                           rgg_update_result *res, int)
{
    labels_body<R>(rm, labels, gray, cap, res);
}

__global__ void __launch_bounds__(kBlock) k_count(RmDev rm)
{
    count_body(rm, (int)blockIdx.x);
}

__global__ void __launch_bounds__(kBlock) k_write(RmDev rm, uint8_t *labels, int64_t *gray, int64_t cap,
                                                  rgg_update_result *res, int force)
{
    write_body(rm, labels, gray, cap, res, force, (int)blockIdx.x);
}

// ------------------------------------------------------------------------
// batched updates of distinct roadmaps: one launch per stage for all of
// them; each kernel finds its request in the device table
// ------------------------------------------------------------------------

// Copies a table row (or its device view) into LDS, all threads, barriers
// around.  One round of vector loads replaces the chain of scalar loads the
// compiler would otherwise issue field by field as the kernel needs them
// (each waiting on the one before, since the view holds the pointers).
template <typename R>
__device__ inline void load_row(R *dst, const R &src)
{
    static_assert(sizeof(R) % 4 == 0, "a row is copied as 32-bit words");
    __syncthreads();
    const uint32_t *a = reinterpret_cast<const uint32_t *>(&src);
    uint32_t *b = reinterpret_cast<uint32_t *>(dst);
    for (int k = threadIdx.x; k < (int)(sizeof(R) / 4); k += blockDim.x) b[k] = a[k];
    __syncthreads();
}

// A row of the table as the item kernel reads it: in constant memory for the
// compiler (no kernel after the diff writes the table), so that the view's
// fields are scalar loads into scalar registers, as a single update's kernel
// arguments are.  From a copy in LDS every field took vector registers, which
// this kernel has none to spare of: 116 B of spills per lane in 2-D and 196 in
// 3-D against 52 and 132 now, 16 planar roadmaps 71.4 -> 66.6 us, 12 spatial
// ones 161 -> 153.  (With three blocks per CU and no spills small batches
// would gain 1 to 4 us more, but 20 roadmaps of up to 12k nodes lose 4 to 11.)
__device__ __forceinline__ const RmDev &const_row(const RmDev &rm)
{
    typedef const __attribute__((address_space(4))) RmDev *Ptr;
    return *(const RmDev *)(Ptr)(uintptr_t)&rm;
}

// One block per roadmap.  With h_tab (this launch's pinned host rows) the
// block reads its row from host memory and writes it to the device table,
// where the later stages read it.
__global__ void __launch_bounds__(kDiffBlock) k_diff_batch(BatchReq *tab, const BatchReq *h_tab)
{
    __shared__ BatchReq q;
    if (h_tab) {
        load_row(&q, h_tab[blockIdx.x]);
        const uint32_t *a = reinterpret_cast<const uint32_t *>(&q);
        uint32_t *b = reinterpret_cast<uint32_t *>(&tab[blockIdx.x]);
        for (int k = threadIdx.x; k < (int)(sizeof(BatchReq) / 4); k += blockDim.x) b[k] = a[k];
    } else {
        load_row(&q, tab[blockIdx.x]);
    }
    // a grid's cells are activated here: a batch has many items to choose from
    const int32_t fixed = q.rm.ncells == 1 ? q.rm.n_fixed : 0;
    if (q.rm.D == 3) diff_body<3>(q.rm, q.a.old_b, q.a.new_b, fixed);
    else diff_body<2>(q.rm, q.a.old_b, q.a.new_b, fixed);
}

// The items of all requests of one group form one range: request r owns
// [P_r, P_r + n_items_r).  Block b of G takes items b, b + G, ..., up to
// kBatchStatic of them, then claims the rest one at a time from a counter
// (items kBatchStatic * G on), so blocks whose items were light take more
// and the launch ends near the mean block time rather than the heaviest
// block's.  The next claim is issued before the current item runs, so its
// latency is hidden.
template <int D, typename T>
__device__ __forceinline__ void item_batch_body(const BatchReq *tab, const int32_t *grp, int n)
{
    __shared__ int s_pref[kMaxBatch + 1];
    __shared__ int s_w[kWaves];
    __shared__ int s_next;
    const int tid = threadIdx.x;
    int v = 0;
    if (tid < n) {
        const RmDev &rm = tab[grp[tid]].rm;
        v = rm.ctl->status == RGG_OK ? min(rm.ctl->n_items, (int32_t)rm.items_cap) : 0;
    }
    int tot;
    const int pre = block_scan(v, &tot, s_w);
    if (tid < n) s_pref[tid] = pre;
    if (tid == 0) s_pref[n] = tot;
    __syncthreads();
    const int G = (int)gridDim.x;
    int32_t *const claim = &tab[grp[0]].rm.ctl->claim;   // reset by the diff of this update
    int g = (int)blockIdx.x;
    for (int k = 0; g < tot; ++k) {
        // the request owning item g: the last r with s_pref[r] <= g (uniform)
        int lo = 0, hi = n - 1;
        while (lo < hi) {
            const int mid = (lo + hi + 1) >> 1;
            if (s_pref[mid] <= g) lo = mid;
            else hi = mid - 1;
        }
        const bool claims = k + 1 >= kBatchStatic;
        int nxt = 0;
        if (claims && tid == 0) nxt = kBatchStatic * G + atomicAdd(claim, 1);
        const int li = __builtin_amdgcn_readfirstlane(g - s_pref[lo]);
        item_body<D, T, 0, false, true>(const_row(tab[__builtin_amdgcn_readfirstlane(grp[lo])].rm), li, 1, false);
        if (claims && tid == 0) s_next = nxt;
        __syncthreads();
        g = claims ? s_next : g + G;
    }
}

template <int D>
__global__ void __launch_bounds__(kBlock, 4) k_item32_batch(const BatchReq *tab, const int32_t *grp, int n)
{
    item_batch_body<D, float>(tab, grp, n);
}

template <int D>
__global__ void __launch_bounds__(kBlock) k_item64_batch(const BatchReq *tab, const int32_t *grp, int n)
{
    item_batch_body<D, double>(tab, grp, n);
}

// request owning a tile: the last r with first[r] <= tile (n <= kMaxBatch)
__device__ inline int owner_of(const BatchReq *tab, int n, int tile, bool write_tiles)
{
    __shared__ int s_r;
    if (threadIdx.x < 64) {
        int best = -1;
        for (int r = threadIdx.x; r < n; r += 64) {
            const int f = write_tiles ? tab[r].wtile0 : tab[r].tile0;
            if (f <= tile) best = max(best, r);
        }
        for (int o = 32; o > 0; o >>= 1) best = max(best, __shfl_xor(best, o));
        if (threadIdx.x == 0) s_r = best;
    }
    __syncthreads();
    return s_r;
}

// The batch's two label passes.  The first writes the labels as it counts
// a tile's GRAY edges (when the update succeeded and the caller asked for
// labels), so the second reads one byte per edge instead of the 8-byte
// counters to place the GRAY ids.
__global__ void __launch_bounds__(kBlock) k_count_batch(const BatchReq *tab, int n)
{
    __shared__ int s_w[kWaves];
    __shared__ BatchReq q;
    const int r = owner_of(tab, n, (int)blockIdx.x, false);
    load_row(&q, tab[r]);
    const RmDev &rm = q.rm;
    const int tile = (int)blockIdx.x - q.tile0;
    const int tid = threadIdx.x;
    const int64_t e0 = (int64_t)tile * kLabelTile + (int64_t)tid * kLabelRun;
    const int status = rm.ctl->status;   // issued before the counters' loads are waited on
    uint8_t lab[kLabelRun];
    const int ng = run_labels(rm, e0, lab);
    if (status == RGG_OK) store_run(rm, q.a.labels, e0, lab);
    const int tot = block_sum(ng, s_w);
    if (tid == 0) rm.tile_cnt[tile] = tot;
}

// A run's labels as k_count_batch wrote them.
__device__ __forceinline__ int load_labels(const RmDev &rm, const uint8_t *labels, int64_t e0,
                                           uint8_t (&lab)[kLabelRun])
{
    if (e0 + kLabelRun <= rm.E && ((uintptr_t)(labels + e0) & 15u) == 0) {
        const uint4 v = *reinterpret_cast<const uint4 *>(labels + e0);
        const uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
        for (int h = 0; h < kLabelRun; ++h) lab[h] = (uint8_t)(w[h >> 2] >> (8 * (h & 3)));
    } else {
#pragma unroll
        for (int h = 0; h < kLabelRun; ++h) lab[h] = e0 + h < rm.E ? labels[e0 + h] : (uint8_t)RGG_GREEN;
    }
    int ng = 0;
#pragma unroll
    for (int h = 0; h < kLabelRun; ++h) ng += (e0 + h < rm.E && lab[h] == RGG_GRAY) ? 1 : 0;
    return ng;
}

__global__ void __launch_bounds__(kBlock) k_write_batch(const BatchReq *tab, int n)
{
    __shared__ BatchReq q;
    const int r = owner_of(tab, n, (int)blockIdx.x, true);
    load_row(&q, tab[r]);
    const int tile = (int)blockIdx.x - q.wtile0;
    if (!q.a.labels || tile == q.rm.ntiles) {
        write_body(q.rm, q.a.labels, q.a.gray, q.a.gray_cap, q.a.res, 0, tile);
        return;
    }
    // the labels are written: the GRAY ids from them
    __shared__ int s_w[kWaves];
    const RmDev &rm = q.rm;
    const int tid = threadIdx.x;
    // the labels and the earlier tiles' counts are loaded with the status,
    // not after it (unused when the update failed)
    const int status = rm.ctl->status;
    int before = 0;
    for (int t = tid; t < tile; t += kBlock) before += rm.tile_cnt[t];
    const int64_t e0 = (int64_t)tile * kLabelTile + (int64_t)tid * kLabelRun;
    uint8_t lab[kLabelRun];
    const int ng = load_labels(rm, q.a.labels, e0, lab);
    if (tid == 0 && tile == 0 && q.a.res) {
        q.a.res->status = status;
        q.a.res->n_changed = rm.ctl->n_chg;
        if (status != RGG_OK) q.a.res->n_gray = 0;
    }
    if (status != RGG_OK) return;
    before = block_sum(before, s_w);
    int tot;
    const int pre = block_scan(ng, &tot, s_w);
    if (tid == 0 && tile == rm.ntiles - 1 && q.a.res) q.a.res->n_gray = (int64_t)before + tot;
    if (tot == 0) return;
    store_gray(rm, q.a.gray, q.a.gray_cap, e0, lab, before, pre, tot);
}

}  // namespace

namespace {

// The kernel of role k for the roadmap's dimension and form: 0 the item kernel
// and 1 the pair testing of the FP32 mode with pair listing, 2 the item kernel
// of the FP64 mode, 3 and 4 that of the FP32 mode without listing (4: few items).
template <int D, int MODE>
void *fn_of(int k)
{
    switch (k) {
    case 0: return (void *)k_item32<D, MODE, true, 4>;
    case 1: return (void *)k_pairs<D, MODE>;
    case 3: return (void *)k_item32<D, MODE, false, 4>;
    case 4: return (void *)k_item32<D, MODE, false, kRoomyPerCu>;
    default: return (void *)k_item64<D, MODE>;   // 2
    }
}

template <int D>
void *fn_dim(int mode, int k)
{
    switch (mode) {
    case kModeObb: return fn_of<D, kModeObb>(k);
    case kModeSplines: return fn_of<D, kModeSplines>(k);
    case kModeObb | kModeSplines: return fn_of<D, kModeObb | kModeSplines>(k);
    default: return fn_of<D, 0>(k);
    }
}

void *fn(const RmDev &rm, int k) { return rm.D == 3 ? fn_dim<3>(rm.mode, k) : fn_dim<2>(rm.mode, k); }


// Label tiles from which k_labels runs in blocks of 1,024 threads: the loads of
// a tile's counters then come 2 KB in a row per wavefront instead of 128 bytes
// apart per lane, at the price of a larger block's barriers.  Updates of planar
// edges with blocks of 256 and of 1,024: 1 tile 24.0 / 24.8 us, 2: 25.8 / 26.0,
// 4: 24.8 / 24.8, 8: 24.7 / 24.8, 12: 25.7 / 25.4, 15: 25.4 / 24.9, 20: 25.6 /
// 25.5, 40: 26.6 / 26.4; spatial ones cross between 8 and 12 tiles too (71
// tiles: 39.0 / 38.4), the arm's between 12 (38.9 / 39.2) and 14 (36.8 / 36.9).
constexpr int kWideTiles = 12;

struct Node {
    void *fn;
    dim3 grid;
    int kind;      // argument list: 0 diff, 1 (rm) only, 4 labels (5: in wide blocks)
    int ev0, ev1;  // stage events ev[ev0..ev1] are recorded after the node
};

// The kernels of one update, in order.  Stage events: ev[0] before, ev[1]
// after the diff, ev[2] after the cell activation, ev[3] after the FP32 item
// kernel, ev[4] after the pair testing, ev[5] after the binary64 re-test (part
// of the two before it: no time), ev[6] after the labels.  The FP64 mode's one
// item kernel stands for the testing (ev[3] before it).
// Blocks of the item kernel for fixed items: one per item, at most kGrid.
unsigned fixed_items_grid(const RmDev &rm) { return (unsigned)std::max(1, std::min(kGrid, rm.n_fixed)); }

int plan(const RmDev &rm, Node out[7])
{
    int n = 0;
    const bool fixed = rm.n_fixed > 0;
    void *const diff_fn = rm.D == 3 ? (void *)k_diff<3> : (void *)k_diff<2>;
    if (rm.mixed) {
        out[n++] = {diff_fn, dim3(1), 0, 1, 2};
        // with every round tested inline there is nothing to share out
        const bool share = rm.inline_rounds != kInlineAll;
        // blocks past the fixed items would only start and stop (with pair
        // listing every block writes its list's count, so the whole grid runs)
        const unsigned grid = fixed && !share ? fixed_items_grid(rm) : kGrid;
        const bool roomy = fixed && rm.n_fixed <= rm.roomy_items;
        out[n++] = {fn(rm, share ? 0 : (roomy ? 4 : 3)), dim3(grid), 1, 3, share ? 3 : 5};
        if (share) out[n++] = {fn(rm, 1), dim3(kGrid), 1, 4, 5};
    } else {
        out[n++] = {diff_fn, dim3(1), 0, 1, 3};
        out[n++] = {fn(rm, 2), dim3(fixed ? fixed_items_grid(rm) : kGrid), 1, 4, 5};
    }
    const bool wide = rm.ntiles >= kWideTiles;
    out[n++] = {wide ? (void *)k_labels<kWideRun> : (void *)k_labels<kLabelRun>, dim3(rm.ntiles + 1), wide ? 5 : 4, 6, 6};
    return n;
}

// kernel arguments of one node (storage for the values lives in `Args`)
struct Args {
    RmDev r;
    const rgg_box *ob, *nb;
    uint8_t *lab;
    int64_t *gray;
    int64_t cap;
    rgg_update_result *res;
    int zero = 0;
    void *diff[3], *one[1], *write[6];
    Args(const RmDev &rm, const UpdateArgs &a)
        : r(rm), ob(a.old_b), nb(a.new_b), lab(a.labels), gray(a.gray), cap(a.gray_cap), res(a.res),
          diff{&r, (void *)&ob, (void *)&nb}, one{&r},
          write{&r, &lab, &gray, &cap, &res, &zero}
    {
    }
    Args(const Args &) = delete;
    void **of(int kind)
    {
        return kind == 0 ? diff : (kind >= 4 ? write : one);
    }
    dim3 block(int kind) const
    {
        return dim3(kind == 0 ? kDiffBlock : (kind == 5 ? kLabelTile / kWideRun : kBlock));
    }
};

}  // namespace

hipError_t launch_marked(const void *fn, dim3 grid, dim3 block, void **args, hipStream_t s, hipEvent_t done,
                         unsigned lds_bytes)
{
    if (!done) return hipLaunchKernel(fn, grid, block, args, lds_bytes, s);
    hipStreamCaptureStatus cs = hipStreamCaptureStatusNone;
    const hipError_t q = hipStreamIsCapturing(s, &cs);
    if (q == hipSuccess && cs == hipStreamCaptureStatusNone)
        return hipExtLaunchKernel(fn, grid, block, args, lds_bytes, s, nullptr, done, 0);
    if (q != hipSuccess) (void)hipGetLastError();
    const hipError_t err = hipLaunchKernel(fn, grid, block, args, lds_bytes, s);
    return err != hipSuccess ? err : hipEventRecord(done, s);
}

hipError_t launch_update(const RmDev &rm, const UpdateArgs &a, hipStream_t s, hipEvent_t *ev, hipEvent_t done)
{
    if (rm.chunk < 1 || rm.chunk > kItemCap) return hipErrorInvalidValue;   // at most kSlots edges of an item per thread
    Node nodes[7];
    const int n = plan(rm, nodes);
    Args args(rm, a);
    hipError_t err;
    if (ev && (err = hipEventRecord(ev[0], s)) != hipSuccess) return err;
    for (int k = 0; k < n; ++k) {
        const Node &nd = nodes[k];
        if ((err = launch_marked(nd.fn, nd.grid, args.block(nd.kind), args.of(nd.kind), s,
                                 k + 1 == n ? done : nullptr)) != hipSuccess)
            return err;
        if (ev && nd.ev0 >= 0)
            for (int m = nd.ev0; m <= nd.ev1; ++m)
                if ((err = hipEventRecord(ev[m], s)) != hipSuccess) return err;
    }
    return hipSuccess;
}

int update_kernels(const RmDev &rm)
{
    Node nodes[7];
    return plan(rm, nodes);
}

int item_edges_max() { return kItemCap; }

__global__ void __launch_bounds__(kBlock) k_cell_slots(RmDev rm, int4 *out, int64_t n)
{
    const int64_t k = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (k >= n) return;
    const int e = rm.cell_edges[k];
    const int jfix = rm.p_fixed ? rm.p_fixed / rm.B : 0;
    int j0, J;
    if (jfix) {
        J = jfix;
        j0 = (int)(uint32_t)((int64_t)e * jfix);
    } else {
        const int64_t s0 = rm.soff[e];
        j0 = (int)(uint32_t)(s0 / rm.B);
        J = (int)((rm.soff[e + 1] - s0) / rm.B);
    }
    out[k] = make_int4(e, j0, J, 0);
}

hipError_t fill_cell_slots(const RmDev &rm, int4 *out, int64_t n, hipStream_t s)
{
    if (n <= 0) return hipSuccess;
    k_cell_slots<<<dim3((unsigned)((n + kBlock - 1) / kBlock)), dim3(kBlock), 0, s>>>(rm, out, n);
    return hipGetLastError();
}

hipError_t test_blocks_resident(int D, int device, int *out)
{
    int per_cu = 0, n_cu = 0;
    hipError_t e = D == 3 ? hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, k_pairs<3, 0>, kBlock, 0)
                          : hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, k_pairs<2, 0>, kBlock, 0);
    if (e != hipSuccess) return e;
    if ((e = hipDeviceGetAttribute(&n_cu, hipDeviceAttributeMultiprocessorCount, device)) != hipSuccess) return e;
    *out = per_cu * n_cu;
    return hipSuccess;
}

hipError_t item_blocks_resident(int D, int device, int *out)
{
    int per_cu = 0, n_cu = 0;
    hipError_t e = D == 3 ? hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, k_item32<3, 0, true, 4>, kBlock, 0)
                          : hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, k_item32<2, 0, true, 4>, kBlock, 0);
    if (e != hipSuccess) return e;
    if ((e = hipDeviceGetAttribute(&n_cu, hipDeviceAttributeMultiprocessorCount, device)) != hipSuccess) return e;
    *out = per_cu * n_cu;
    return hipSuccess;
}

hipError_t launch_labels(const RmDev &rm, const UpdateArgs &a, hipStream_t s)
{
    k_count<<<rm.ntiles, kBlock, 0, s>>>(rm);
    hipError_t err = hipGetLastError();
    if (err != hipSuccess) return err;
    k_write<<<rm.ntiles, kBlock, 0, s>>>(rm, a.labels, a.gray, a.gray_cap, a.res, 1);
    return hipGetLastError();
}

hipError_t add_update_nodes(hipGraph_t g, const RmDev &rm, const UpdateArgs &a, hipGraphNode_t dep,
                            hipGraphNode_t *last)
{
    if (rm.chunk < 1 || rm.chunk > kItemCap) return hipErrorInvalidValue;
    Node nodes[7];
    const int n = plan(rm, nodes);
    Args args(rm, a);   // hipGraphAddKernelNode copies the argument values
    hipGraphNode_t prev = dep;
    for (int k = 0; k < n; ++k) {
        hipKernelNodeParams p = {};
        p.func = nodes[k].fn;
        p.gridDim = nodes[k].grid;
        p.blockDim = args.block(nodes[k].kind);
        p.sharedMemBytes = 0;
        p.kernelParams = args.of(nodes[k].kind);
        p.extra = nullptr;
        hipGraphNode_t node;
        hipError_t err = hipGraphAddKernelNode(&node, g, prev ? &prev : nullptr, prev ? 1 : 0, &p);
        if (err != hipSuccess) return err;
        prev = node;
    }
    *last = prev;
    return hipSuccess;
}

namespace {

// The kernels of a batched update in order, each handed to `emit(fn, grid,
// block, args)` (a graph-node adder or a stream launcher).  With `h_tab`
// (pinned host rows) the diff kernel copies them to `tab`, so a launch needs no
// copy engine, whose hand-over to the kernels' queue costs more than the copy.
// `after(stage)` follows each kernel: 0 diff, 1 cells, 3 item, 5 labels (count
// and write).
template <typename Emit, typename After>
hipError_t batch_kernels(Emit emit, After after, const BatchReq *tab, const BatchReq *h_tab, const int32_t *grp,
                         int n, const BatchGroup *groups, int n_groups, bool any_grid, int n_tiles, int n_wtiles)
{
    const BatchReq *t = tab;
    int nn = n;
    hipError_t err;
    BatchReq *t_dst = const_cast<BatchReq *>(tab);
    const BatchReq *t_src = h_tab;
    void *a_first[] = {(void *)&t_dst, (void *)&t_src};
    if ((err = emit((void *)k_diff_batch, dim3(n), dim3(kDiffBlock), a_first)) != hipSuccess) return err;
    void *a_diff[] = {(void *)&t};
    if ((err = after(0)) != hipSuccess) return err;
    void *a_tn[] = {(void *)&t, (void *)&nn};
    // the grid roadmaps' cells are activated by the diff kernel itself
    if (any_grid && (err = after(1)) != hipSuccess) return err;
    for (int k = 0; k < n_groups; ++k) {
        const BatchGroup &gr = groups[k];
        const int32_t *gp = grp + gr.off;
        int cnt = gr.count;
        void *a_item[] = {(void *)&t, (void *)&gp, (void *)&cnt};
        void *fn = gr.D == 3 ? (gr.mixed ? (void *)k_item32_batch<3> : (void *)k_item64_batch<3>)
                             : (gr.mixed ? (void *)k_item32_batch<2> : (void *)k_item64_batch<2>);
        if ((err = emit(fn, dim3(kBatchItemGrid), dim3(kBlock), a_item)) != hipSuccess) return err;
        if ((err = after(3)) != hipSuccess) return err;
    }
    if ((err = emit((void *)k_count_batch, dim3(n_tiles), dim3(kBlock), a_tn)) != hipSuccess) return err;
    if ((err = emit((void *)k_write_batch, dim3(n_wtiles), dim3(kBlock), a_tn)) != hipSuccess) return err;
    return after(5);
}

}  // namespace

hipError_t add_batch_nodes(hipGraph_t g, const BatchReq *tab, const BatchReq *h_tab, const int32_t *grp, int n,
                           const BatchGroup *groups, int n_groups, bool any_grid, int n_tiles,
                           int n_wtiles, hipGraphNode_t dep, hipGraphNode_t *last)
{
    hipGraphNode_t prev = dep;
    auto add = [&](void *fn, dim3 grid, dim3 block, void **args) -> hipError_t {
        hipKernelNodeParams p = {};
        p.func = fn;
        p.gridDim = grid;
        p.blockDim = block;
        p.sharedMemBytes = 0;
        p.kernelParams = args;
        p.extra = nullptr;
        hipGraphNode_t node;
        hipError_t err = hipGraphAddKernelNode(&node, g, prev ? &prev : nullptr, prev ? 1 : 0, &p);
        if (err == hipSuccess) prev = node;
        return err;
    };
    auto none = [](int) { return hipSuccess; };
    hipError_t err = batch_kernels(add, none, tab, h_tab, grp, n, groups, n_groups, any_grid, n_tiles, n_wtiles);
    if (err == hipSuccess) *last = prev;
    return err;
}

// The request table of rgg_update_batch_noalloc.  Host code never passes the
// array's name to a kernel or a copy: it uses the address that
// batch_scratch_address returns for the current device.
static __device__ __align__(256) unsigned char scratch[kBatchScratchBytes];

hipError_t batch_scratch_address(void **ptr)
{
    *ptr = nullptr;
    return hipGetSymbolAddress(ptr, HIP_SYMBOL(scratch));
}

hipError_t launch_batch(hipStream_t s, const BatchReq *tab, const BatchReq *h_tab, const int32_t *grp, int n,
                        const BatchGroup *groups, int n_groups, bool any_grid, int n_tiles, int n_wtiles,
                        BatchTiming *timing, hipEvent_t done)
{
    auto launch = [&](void *fn, dim3 grid, dim3 block, void **args) -> hipError_t {
        // the gray lists' kernel is the batch's last
        return launch_marked(fn, grid, block, args, s, fn == (void *)k_write_batch ? done : nullptr);
    };
    if (!timing) {
        auto none = [](int) { return hipSuccess; };
        return batch_kernels(launch, none, tab, h_tab, grp, n, groups, n_groups, any_grid, n_tiles, n_wtiles);
    }
    timing->n = 0;
    auto mark = [&](int stage) -> hipError_t {
        if (timing->n >= BatchTiming::kMax) return hipErrorInvalidValue;
        timing->stage[timing->n] = stage;
        return hipEventRecord(timing->ev[1 + timing->n++], s);
    };
    hipError_t err = hipEventRecord(timing->ev[0], s);
    if (err != hipSuccess) return err;
    return batch_kernels(launch, mark, tab, h_tab, grp, n, groups, n_groups, any_grid, n_tiles, n_wtiles);
}

}  // namespace rgg
