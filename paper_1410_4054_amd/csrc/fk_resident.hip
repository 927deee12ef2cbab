// Resident solvers: a whole pipelined solve in one launch of at most one
// workgroup per compute unit, for systems whose matrix and vectors fit the
// registers and LDS of the chip.  (arXiv:1410.4054, Algorithms 2 and 4; the
// same iterates as the kernels of fk_kernels.hip.)
//
// Why.  Below about a million unknowns an iteration of the launch-per-step
// kernels is bound by launches, by the two-level second stage of their
// reductions and by reading vectors and matrix back from the caches (2D
// Poisson: 12.3 us per CG iteration at N = 16,129, 18 us at 261,121).  Here
// workgroup g owns `rows` consecutive rows for the whole solve: its part of
// the matrix and its x, r, A p stay in registers, p in LDS, and one hand-over
// between workgroups per product is left.
//
// Ghosts.  The columns a workgroup's rows reach outside its own rows are its
// ghosts (k_res_plan lists them once per solver and rewrites every entry's
// column as a 16-bit index into [own rows | ghosts]).  A workgroup keeps r
// and p of its ghosts too and updates them itself, with the owner's
// expressions on the owner's operands, so bit for bit the owner's values;
// all it needs from the owner is A p, once per iteration.
//
// Hand-over.  A p of the rows that are somebody's ghost, and the workgroup's
// double-double partials of the inner products, travel as 8-byte words of
// 32 bits of data and a 32-bit tag (the number of the product, never used
// twice in a workspace), stored and read at agent scope (coherent across the
// XCDs).  An 8-byte word arrives whole, so a reader polls the word itself:
// no flags, no fences, nothing to clear.  Words are double-buffered by the
// tag's parity: the owner rewrites a word two products later, after a
// reduction to which every reader has contributed since it read the word.
// Every workgroup reads all partials and adds them in the same fixed tree,
// so all take the same decisions, and one hand-over replaces the grid's
// group leaders, top leader and the next launch's state read.
//
// Residency.  The workgroups wait for one another, so all must be on the
// chip at once.  A launch first agrees on that: workgroups report, workgroup
// 0 decides with one compare-and-swap, anyone who waits too long decides
// against.  Decided against, every workgroup ends with nothing written and
// the host runs the launch-per-step kernels instead.  Later waits are
// bounded too (FK_RES_SPIN_LIMIT polls, seconds): running out marks the
// solve void, as a reduction point does.
#include "fk_dd.hpp"
#include "fk_internal.hpp"
#include "fk_state.hpp"

namespace fk {
namespace {

#ifndef FK_RES_SPIN_LIMIT
#define FK_RES_SPIN_LIMIT (1 << 22)
#endif
// Polls before the launch is given up (about 20 ms).
#ifndef FK_RES_START_LIMIT
#define FK_RES_START_LIMIT (1 << 15)
#endif

constexpr int PLAN_T = 512;
constexpr uint32_t RES_NONE = 0xffffu;  // no entry

// ------------------------------------------------------------------ plan

// Column of entry k of row `row` in slice sl (e0 its first entry), -1: none.
__device__ __forceinline__ int entry_col(const DevCsr &A, int sl, int e0, int k, int lane, int row)
{
    if (A.dg_mask)
        return (A.dg_mask[row] >> k & 1u) ? row + A.dg_off[e0 / SLICE + k] : -1;
    if (A.sell_off4) {
        const short4 o = A.sell_off4[A.sell_ptr4[sl] + (k / 4) * SLICE + lane];
        const int16_t v = (k & 3) == 0 ? o.x : (k & 3) == 1 ? o.y : (k & 3) == 2 ? o.z : o.w;
        return v == SELL_PAD ? -1 : row + (int)v;
    }
    return A.sell_col[e0 + k * SLICE + lane];
}

// Workgroup g: its ghosts in ascending order (at most gcap of them are
// stored), their number (-1: the columns span more than the bitmap) and the
// 16-bit index of every entry of its slices; pub[c] = 1 for every ghost c.
// Slice j of workgroup g is perm[g * spw + j] (-1: none); owner[slice] =
// g << 16 | j.
__global__ __launch_bounds__(PLAN_T) void k_res_plan(DevCsr A, int spw, int gcap, const int32_t *perm,
                                                     const int32_t *owner, uint16_t *idx, int32_t *gcount,
                                                     int32_t *glist, uint8_t *pub)
{
    __shared__ uint32_t bits[RES_PLAN_WORDS];
    __shared__ uint32_t pre[PLAN_T];
    __shared__ int lo_s, hi_s;
    const int g = blockIdx.x, tid = threadIdx.x, lane = tid & 63;
    // f(entry, column or -1, local slice) over the workgroup's entries
    auto entries = [&](auto &&f) {
        for (int j = tid / 64; j < spw; j += PLAN_T / 64) {
            const int sl = perm[g * spw + j];
            if (sl < 0)
                continue;
            const int e0 = A.sell_ptr[sl], width = (A.sell_ptr[sl + 1] - e0) / SLICE, row = sl * SLICE + lane;
            for (int k = 0; k < width; ++k)
                f(e0 + k * SLICE + lane, row < A.n ? entry_col(A, sl, e0, k, lane, row) : -1);
        }
    };
    auto mine = [&](int c) { return owner[c / SLICE] >> 16 == g; };
    if (tid == 0) {
        lo_s = A.n;
        hi_s = -1;
    }
    __syncthreads();
    int lo = A.n, hi = -1;
    entries([&](int, int c) {
        if (c >= 0 && !mine(c)) {
            lo = min(lo, c);
            hi = max(hi, c);
        }
    });
    atomicMin(&lo_s, lo);
    atomicMax(&hi_s, hi);
    __syncthreads();
    lo = lo_s;
    const int64_t span = max((int64_t)hi_s - lo + 1, (int64_t)0);
    if (span > (int64_t)RES_PLAN_WORDS * 32) {
        if (tid == 0)
            gcount[g] = -1;
        return;
    }
    const int nw = (int)((span + 31) / 32);
    for (int w = tid; w < nw; w += PLAN_T)
        bits[w] = 0;
    __syncthreads();
    entries([&](int, int c) {
        if (c >= 0 && !mine(c))
            atomicOr(&bits[(c - lo) >> 5], 1u << ((c - lo) & 31));
    });
    __syncthreads();
    // ghosts before each thread's share of the bitmap
    const int per = (nw + PLAN_T - 1) / PLAN_T;
    const int w0 = min(nw, tid * per), w1 = min(nw, w0 + per);
    uint32_t cnt = 0;
    for (int w = w0; w < w1; ++w)
        cnt += __popc(bits[w]);
    pre[tid] = cnt;
    __syncthreads();
    for (int s = 1; s < PLAN_T; s <<= 1) {
        const uint32_t v = tid >= s ? pre[tid - s] : 0;
        __syncthreads();
        pre[tid] += v;
        __syncthreads();
    }
    if (tid == 0)
        gcount[g] = (int)pre[PLAN_T - 1];
    uint32_t at = pre[tid] - cnt;
    for (int w = w0; w < w1; ++w) {
        for (uint32_t m = bits[w]; m; m &= m - 1) {
            const int c = lo + w * 32 + __builtin_ctz(m);
            pub[c] = 1;
            if ((int)at < gcap)
                glist[(size_t)g * gcap + at] = c;
            ++at;
        }
    }
    entries([&](int e, int c) {
        uint32_t v = RES_NONE;
        if (c >= 0 && mine(c)) {
            v = (uint32_t)((owner[c / SLICE] & 0xffff) * SLICE + c % SLICE);
        } else if (c >= 0) {
            const int w = (c - lo) >> 5, t = w / per;
            uint32_t r = t > 0 ? pre[t - 1] : 0;
            for (int u = t * per; u < w; ++u)
                r += __popc(bits[u]);
            r += __popc(bits[w] & ((1u << ((c - lo) & 31)) - 1u));
            v = (uint32_t)(spw * SLICE) + r;
        }
        idx[e] = (uint16_t)v;
    });
}

// Streamed matrices: the indices of a row's entries as four words of two
// (pads and missing entries: the gathered vector's zero).
__global__ __launch_bounds__(256) void k_res_pack(DevCsr A, int rows, const int32_t *owner, const int32_t *gcount,
                                                  const uint16_t *idx, uint4 *out)
{
    const int sl = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
    if (sl >= A.nslices)
        return;
    const int e0 = A.sell_ptr[sl], width = (A.sell_ptr[sl + 1] - e0) / SLICE;
    const uint32_t zero = (uint32_t)(rows + 2 * gcount[owner[sl] >> 16]);
    uint32_t w[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) {
        const uint32_t i = k < width ? idx[e0 + k * SLICE + lane] : RES_NONE;
        w[k] = i == RES_NONE ? zero : i;
    }
    out[(size_t)sl * SLICE + lane] =
        uint4{w[0] | w[1] << 16, w[2] | w[3] << 16, w[4] | w[5] << 16, w[6] | w[7] << 16};
}

// ------------------------------------------------------------- hand-over

__device__ __forceinline__ uint64_t load_word(const uint64_t *p)
{
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

__device__ __forceinline__ void store_word(uint64_t *p, uint32_t tag, uint32_t half)
{
    __hip_atomic_store(p, (uint64_t)tag << 32 | half, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// A double as two tagged words.
__device__ __forceinline__ void store_tagged(uint64_t *p, uint32_t tag, double v)
{
    const uint64_t b = (uint64_t)__double_as_longlong(v);
    store_word(p, tag, (uint32_t)b);
    store_word(p + 1, tag, (uint32_t)(b >> 32));
}

__device__ __forceinline__ bool tagged(uint64_t lo, uint64_t hi, uint32_t tag)
{
    return (uint32_t)(lo >> 32) == tag && (uint32_t)(hi >> 32) == tag;
}

__device__ __forceinline__ double untag(uint64_t lo, uint64_t hi)
{
    return __longlong_as_double((long long)((uint64_t)(uint32_t)lo | hi << 32));
}

// Sums of four double-doubles over the lanes at once.  A tree per dot adds
// in every lane at every level, four trees of six levels; here the first
// two levels also deal the dots out: lane l ends with dot l & 3 (2 + 1
// additions), and the further levels add one value per lane.
template <int CTRL>
__device__ __forceinline__ dd dpp_dd(dd v)
{
    return dd{dpp_double<CTRL, 0xf>(v.hi), dpp_double<CTRL, 0xf>(v.lo)};
}

__device__ __forceinline__ dd pick(bool c, dd a, dd b) { return dd{c ? a.hi : b.hi, c ? a.lo : b.lo}; }

// Lane l: dot l & 3 summed over the four lanes of its quad.
template <int K>
__device__ __forceinline__ dd deal(const dd (&v)[K])
{
    const bool b0 = threadIdx.x & 1, b1 = threadIdx.x & 2;
    constexpr int XOR1 = 0xb1, XOR2 = 0x4e;  // quad_perm [1,0,3,2], [2,3,0,1]
    const dd a = dd_add(pick(b0, v[1], v[0]), dpp_dd<XOR1>(pick(b0, v[0], v[1])));
    dd b{0.0, 0.0};
    if constexpr (K > 2) {
        const dd z{0.0, 0.0};
        const dd v3 = K > 3 ? v[K - 1] : z;
        b = dd_add(pick(b0, v3, v[2]), dpp_dd<XOR1>(pick(b0, v[2], v3)));
    }
    return dd_add(pick(b1, b, a), dpp_dd<XOR2>(pick(b1, a, b)));
}

// Lane l: the sum over the lanes of its row of 16 with the same l & 3
// (rotations: every such lane adds the same values in a commuted order, and
// dd_add commutes bit for bit).
__device__ __forceinline__ dd row_quads(dd v)
{
    v = dd_add(v, dpp_dd<0x128>(v));  // row_ror:8
    return dd_add(v, dpp_dd<0x124>(v));  // row_ror:4
}

// ... and over the four rows.
__device__ __forceinline__ void swap_rows16(double x, double &a, double &b)
{
    const uint64_t u = (uint64_t)__double_as_longlong(x);
    const auto lo = __builtin_amdgcn_permlane16_swap((uint32_t)u, (uint32_t)u, false, false);
    const auto hi = __builtin_amdgcn_permlane16_swap((uint32_t)(u >> 32), (uint32_t)(u >> 32), false, false);
    a = __longlong_as_double((long long)((uint64_t)hi[0] << 32 | lo[0]));
    b = __longlong_as_double((long long)((uint64_t)hi[1] << 32 | lo[1]));
}

__device__ __forceinline__ void swap_rows32(double x, double &a, double &b)
{
    const uint64_t u = (uint64_t)__double_as_longlong(x);
    const auto lo = __builtin_amdgcn_permlane32_swap((uint32_t)u, (uint32_t)u, false, false);
    const auto hi = __builtin_amdgcn_permlane32_swap((uint32_t)(u >> 32), (uint32_t)(u >> 32), false, false);
    a = __longlong_as_double((long long)((uint64_t)hi[0] << 32 | lo[0]));
    b = __longlong_as_double((long long)((uint64_t)hi[1] << 32 | lo[1]));
}

__device__ __forceinline__ dd wave_quads(dd v)
{
    v = row_quads(v);
    dd a, b;
    swap_rows16(v.hi, a.hi, b.hi);
    swap_rows16(v.lo, a.lo, b.lo);
    v = dd_add(a, b);
    swap_rows32(v.hi, a.hi, b.hi);
    swap_rows32(v.lo, a.lo, b.lo);
    return dd_add(a, b);
}

// A sum that is complete here, with many rows per thread: without this the
// compiler moves the additions of a whole phase to where the sum is used and
// holds every summand (16 rows: 96 registers spilled; none with it).  With
// few rows the moved additions fill the gathers' latency.
template <bool BIG>
__device__ __forceinline__ void settle(dd &v)
{
    if constexpr (BIG)
        asm volatile("" : "+v"(v.hi), "+v"(v.lo));
}

struct ResShared {
    DevState s;
    dd rows[32][4];  // per row of 16 lanes of each wave: the four dots
    dd psum[RES_MAX_WG / 64][4];
    double alpha, beta, omega, rr_next;
    int status;
    int fault;
    int go;
};

// Ghost words a thread holds while the reduction runs: the first GPT ghosts
// of its share (ghost j belongs to thread j % T).
constexpr int GPT = 4;
struct GhostWords {
    uint64_t lo[GPT], hi[GPT];
};

template <int T, bool CLEAR = false>
__device__ __forceinline__ void ghost_load(const uint64_t *ll, const int32_t *gl, int ng, GhostWords &w, int j0 = 0)
{
#pragma unroll
    for (int i = 0; i < GPT; ++i) {
        const int j = j0 + (int)threadIdx.x + i * T;
        if constexpr (CLEAR)
            w.lo[i] = w.hi[i] = 0;  // (nothing held from the last time)
        if (j < ng) {
            const uint64_t *p = ll + 2 * (size_t)gl[j];
            w.lo[i] = load_word(p);
            w.hi[i] = load_word(p + 1);
        }
    }
}

template <int T>
__device__ __forceinline__ bool ghost_ready(int ng, uint32_t tag, const GhostWords &w, int j0 = 0)
{
    bool ok = true;
#pragma unroll
    for (int i = 0; i < GPT; ++i)
        if (j0 + (int)threadIdx.x + i * T < ng)
            ok = ok && tagged(w.lo[i], w.hi[i], tag);
    return ok;
}

// Poll the thread's ghost words until they carry `tag`.
template <int T>
__device__ __forceinline__ bool ghost_poll(const uint64_t *ll, const int32_t *gl, int ng, uint32_t tag, GhostWords &w,
                                           int j0 = 0)
{
    for (int spin = 0; !ghost_ready<T>(ng, tag, w, j0); ++spin) {
        if (spin >= FK_RES_SPIN_LIMIT)
            return false;
        if (spin > 0)
            __builtin_amdgcn_s_sleep(1);
        ghost_load<T>(ll, gl, ng, w, j0);
    }
    return true;
}

// The inner products of all workgroups: v summed over the workgroup,
// published under `tag`, collected (64 workgroups per wave), summed in a
// fixed tree, rounded, and `fin` run on the result by wave 0 of every
// workgroup (all lanes on the same values).  Up to RES_DIRECT workgroups
// every workgroup collects for itself: one hand-over.  Above, workgroup 0
// alone does and hands the rounded sums on: a second hand-over, but 256
// workgroups reading 24 KB each through the fabric take longer than that
// (2D Poisson 255^2, 255 workgroups: 8.9 us per iteration, 6.6 with two).  Waves that
// collect nothing poll the thread's ghost words meanwhile.  Returns false
// when a wait ran out; ends past a barrier.
template <int T, int K, int HALF, typename FIN>
__device__ __forceinline__ bool all_reduce(dd (&v)[K], ResShared &sh, const ResArgs &a, int g, uint32_t tag,
                                           const uint64_t *ll, const int32_t *gl, int ng, GhostWords &gw, FIN &&fin)
{
    constexpr int NR = T / 16;  // rows of 16 lanes
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, dot = lane & 3;
    const int G = gridDim.x;
    const bool direct = G <= RES_DIRECT;
    const int np = direct || g == 0 ? (G + 63) / 64 : 0;  // waves that collect
    // a workgroup's record: four dots of (hi, lo), two words each: 128 bytes
    uint64_t *part = a.part + (size_t)(tag & 1u) * RES_PART_WORDS;
    uint64_t *sums = part + (size_t)16 * RES_MAX_WG;  // the rounded sums, two words each
    {
        const dd r = row_quads(deal(v));
        if ((lane & 15) < 4)
            sh.rows[threadIdx.x >> 4][dot] = r;
    }
    __syncthreads();
    if (wave == 0) {
        dd r = sh.rows[lane >> 2][dot];
        if constexpr (NR > 16)
            r = dd_add(r, sh.rows[16 + (lane >> 2)][dot]);
        r = wave_quads(r);
        if (G == 1) {  // nobody to hand over to
            double d[K];
#pragma unroll
            for (int k = 0; k < K; ++k)
                d[k] = lane_value(r.hi + r.lo, k);
            fin(d);
        } else if (lane < K) {
            store_tagged(part + (size_t)16 * g + 4 * lane, tag, r.hi);
            store_tagged(part + (size_t)16 * g + 4 * lane + 2, tag, r.lo);
        }
    }
    if (G == 1) {
        __syncthreads();
        return true;
    }
    dd mine{0.0, 0.0};
    if (wave < np) {
        // lane: dot l & 3 of the members (l >> 2) + 16 i of the wave's 64, HALF of
        // them at a time (two where registers are short)
        const int m = wave * 64 + (lane >> 2);
        dd q[4];
#pragma unroll
        for (int h = 0; h < 4; h += HALF) {
            uint64_t w[4 * HALF] = {};  // members past G and dots past K: sums of zero
            bool ok = dot >= K;
            for (int spin = 0;; ++spin) {
                if (!ok) {
                    ok = true;
#pragma unroll
                    for (int i = 0; i < HALF; ++i)
                        if (m + 16 * (h + i) < G) {
#pragma unroll
                            for (int j = 0; j < 4; ++j)
                                w[4 * i + j] = load_word(part + (size_t)16 * (m + 16 * (h + i)) + 4 * dot + j);
                        }
#pragma unroll
                    for (int i = 0; i < HALF; ++i)
                        if (m + 16 * (h + i) < G)
                            ok = ok && tagged(w[4 * i], w[4 * i + 1], tag) && tagged(w[4 * i + 2], w[4 * i + 3], tag);
                }
                if (__builtin_amdgcn_ballot_w64(!ok) == 0)
                    break;
                if (spin >= FK_RES_SPIN_LIMIT) {
                    sh.fault = 1;
                    break;
                }
            }
#pragma unroll
            for (int i = 0; i < HALF; ++i)
                q[h + i] = dd{untag(w[4 * i], w[4 * i + 1]), untag(w[4 * i + 2], w[4 * i + 3])};
        }
        ghost_load<T, HALF < 4>(ll, gl, ng, gw);  // in flight during the sums; checked after the last barrier
        mine = wave_quads(dd_add(dd_add(q[0], q[1]), dd_add(q[2], q[3])));
        if (np > 1 && lane < 4)
            sh.psum[wave][dot] = mine;
    } else if (HALF < 4) {
        // (loaded before the first test, so that the last iteration's words need
        // not be held in registers through the product)
        ghost_load<T, true>(ll, gl, ng, gw);
        if (wave > 0 && !ghost_poll<T>(ll, gl, ng, tag, gw))
            sh.fault = 1;
    } else if (wave == 0) {
        ghost_load<T>(ll, gl, ng, gw);
    } else if (!ghost_poll<T>(ll, gl, ng, tag, gw)) {
        sh.fault = 1;
    }
    if (np > 1)
        __syncthreads();
    if (wave == 0) {
        double d[K];
        if (np > 0) {
            if (np > 1)  // lane: dot l & 3 of wave (l >> 2) & 3
                mine = row_quads((lane >> 2 & 3) < np ? sh.psum[lane >> 2 & 3][dot] : dd{0.0, 0.0});
            const double r = mine.hi + mine.lo;
            if (!direct && lane < K)
                store_tagged(sums + 2 * lane, tag, r);
#pragma unroll
            for (int k = 0; k < K; ++k)
                d[k] = lane_value(r, k);
        } else {
            uint64_t w = 0;
            bool ok = lane >= 2 * K;
            for (int spin = 0;; ++spin) {
                if (!ok) {
                    w = load_word(sums + lane);
                    ok = (uint32_t)(w >> 32) == tag;
                }
                if (__builtin_amdgcn_ballot_w64(!ok) == 0)
                    break;
                if (spin >= FK_RES_SPIN_LIMIT) {
                    sh.fault = 1;
                    break;
                }
            }
            const int half = (int)(uint32_t)w;
#pragma unroll
            for (int k = 0; k < K; ++k)
                d[k] = __longlong_as_double((long long)((uint64_t)(uint32_t)__builtin_amdgcn_readlane(half, 2 * k) |
                                                        (uint64_t)(uint32_t)__builtin_amdgcn_readlane(half, 2 * k + 1)
                                                            << 32));
        }
        if (!sh.fault)
            fin(d);
    }
    __syncthreads();
    if (!ghost_poll<T>(ll, gl, ng, tag, gw))
        sh.fault = 1;
    return sh.fault == 0;
}

// All workgroups on the chip: reported, and decided by one compare-and-swap.
template <int T>
__device__ __forceinline__ bool everyone_here(ResShared &sh, const ResArgs &a, int g)
{
    const uint64_t undecided = (uint64_t)a.epoch << 2;
    if (gridDim.x == 1) {
        __syncthreads();
        return true;
    }
    if (threadIdx.x == 0)
        __hip_atomic_store(a.arrived + g, a.epoch, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    bool here = true;
    if (g == 0) {
        bool mine = threadIdx.x >= gridDim.x;
        for (int spin = 0; !mine && spin < FK_RES_START_LIMIT; ++spin) {
            mine = __hip_atomic_load(a.arrived + threadIdx.x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == a.epoch;
            __builtin_amdgcn_s_sleep(1);
        }
        here = __syncthreads_and(mine);
    }
    if (threadIdx.x == 0) {
        uint64_t cur = load_word(a.decision);
        if (g != 0)
            for (int spin = 0; (cur >> 2) != a.epoch && spin < 2 * FK_RES_START_LIMIT; ++spin) {
                __builtin_amdgcn_s_sleep(2);
                cur = load_word(a.decision);
            }
        const uint64_t say = undecided | (g == 0 && here ? 1u : 2u);
        while ((cur >> 2) != a.epoch) {
            const uint64_t seen = atomicCAS(reinterpret_cast<unsigned long long *>(a.decision), cur, say);
            cur = seen == cur ? say : seen;
        }
        sh.go = (cur & 3u) == 1u;
    }
    __syncthreads();
    return sh.go != 0;
}

// -------------------------------------------------------------------- CG

// Index of the thread's row k among the workgroup's.  With four and more rows
// per thread the compiler must not compute what follows from it (addresses,
// unpacked indices of every row) once and hold it over the whole solve: that
// spills the 256 registers.
template <int T, int RPT>
__device__ __forceinline__ int own_row(int k)
{
    int t = threadIdx.x;
    if constexpr (RPT >= 4)
        asm volatile("" : "+v"(t));
    return k * T + t;
}

// Where the values of a row of w entries live.  Eight rows per thread keep
// two of five (three of seven) in LDS, since 256 registers do not hold all
// of them (all in registers: 202 spilled, 1000^2 Poisson 21 us per
// iteration); sixteen rows read them from the caches for every product.
constexpr int ST_AHEAD = 1;  // rows requested ahead (1 to 4 measure alike)
constexpr bool res_streamed(int rpt) { return rpt >= 16; }
constexpr int res_lds_values(int rpt, int w) { return rpt == 8 ? w == 5 ? 2 : 3 : 0; }

// The workgroup's rows of the matrix.  Row k of thread t is row t % 64 of the
// workgroup's slice k T / 64 + t / 64, so a wave holds whole slices.
template <int T, int RPT, int W>
struct ResRows {
    static constexpr bool STREAM = res_streamed(RPT);
    static constexpr int WL = res_lds_values(RPT, W), WR = STREAM ? 0 : W - WL;
    int sl[RPT];  // the slice, -1: none (uniform over the wave)
    [[maybe_unused]] double a[STREAM ? 1 : RPT][WR > 0 ? WR : 1];
    [[maybe_unused]] int ext[STREAM ? RPT : 1];  // streamed: first entry / 64 << 3 | width (uniform)
    double *far;  // values WR .. W-1 of the workgroup's rows, [WL][rows]
    int rows;
    int zero;     // index of an entry of the gathered vector that holds 0
    uint32_t id[STREAM ? 1 : RPT][(W + 1) / 2];  // two 16-bit indices to a word

    __device__ __forceinline__ void load(const ResArgs &r)
    {
        const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x / SLICE)), lane = threadIdx.x & 63;
        const int spw = rows / SLICE;
#pragma unroll
        for (int k = 0; k < RPT; ++k) {
            const int j = k * (T / SLICE) + wave;
            int e0 = 0, width = 0;
            sl[k] = j < spw ? __builtin_amdgcn_readfirstlane(r.perm[blockIdx.x * spw + j]) : -1;
            if (sl[k] >= 0) {
                e0 = __builtin_amdgcn_readfirstlane(r.A.sell_ptr[sl[k]]);
                width = (__builtin_amdgcn_readfirstlane(r.A.sell_ptr[sl[k] + 1]) - e0) / SLICE;
            }
            if constexpr (STREAM) {
                ext[k] = e0 / SLICE << 3 | width;
            } else {
#pragma unroll
                for (int w = 0; w < (W + 1) / 2; ++w)
                    id[k][w] = (uint32_t)zero | (uint32_t)zero << 16;
#pragma unroll
                for (int w = 0; w < W; ++w) {
                    const double v = w < width ? r.A.sell_vals[e0 + w * SLICE + lane] : 0.0;
                    if (w < WR)
                        a[k][w < WR ? w : 0] = v;
                    else if (j < spw)
                        far[(w - WR) * rows + k * T + threadIdx.x] = v;
                    if (w < width) {
                        uint32_t i = r.idx[e0 + w * SLICE + lane];
                        i = i == RES_NONE ? (uint32_t)zero : i;
                        id[k][w / 2] = w & 1 ? (id[k][w / 2] & 0xffffu) | i << 16 : (id[k][w / 2] & 0xffff0000u) | i;
                    }
                }
            }
        }
    }

    // Streamed: request the values and indices of row k.
    __device__ __forceinline__ void request(const ResArgs &r, int k, double (&v)[W], uint4 &i) const
    {
        int e = ext[k], s = sl[k], lane = threadIdx.x & 63;
        asm volatile("" : "+s"(e), "+s"(s));  // see own_row
        asm volatile("" : "+v"(lane));
        const int width = e & 7;
        const double *__restrict__ src = r.A.sell_vals + (size_t)(e >> 3) * SLICE;
        i = uint4{(uint32_t)zero | (uint32_t)zero << 16, (uint32_t)zero | (uint32_t)zero << 16,
                  (uint32_t)zero | (uint32_t)zero << 16, (uint32_t)zero | (uint32_t)zero << 16};
        if (s >= 0)
            i = (r.idx4 + (size_t)s * SLICE)[lane];
        if (width == W) {
#pragma unroll
            for (int w = 0; w < W; ++w)
                v[w] = src[w * SLICE + lane];
        } else {
#pragma unroll
            for (int w = 0; w < W; ++w) {
                v[w] = 0.0;
                if (w < width)
                    v[w] = src[w * SLICE + lane];
            }
        }
    }

    // Row k times v (own rows, then ghosts, then 0), left to right.  A missing
    // entry adds 0 * 0, which changes nothing: the sum starts at +0 and,
    // rounding to nearest, is never -0.
    template <typename VAL>
    __device__ __forceinline__ static double sum(uint32_t (&pair)[(W + 1) / 2], const double *v, VAL &&val)
    {
        double q = 0.0;
#pragma unroll
        for (int w = 0; w < W; ++w) {
            const uint32_t i = w & 1 ? pair[w / 2] >> 16 : pair[w / 2] & 0xffffu;
            q = q + val(w) * v[i];
        }
        return q;
    }
    // f(k, row k times v) for every row, in order.
    template <typename F>
    __device__ __forceinline__ void product(const ResArgs &r, const double *v, F &&f) const
    {
        if constexpr (STREAM) {
            // requested ST_AHEAD rows ahead
            double buf[ST_AHEAD + 1][W];
            uint4 at[ST_AHEAD + 1];
#pragma unroll
            for (int k = 0; k < ST_AHEAD; ++k)
                request(r, k, buf[k], at[k]);
#pragma unroll
            for (int k = 0; k < RPT; ++k) {
                constexpr int M = ST_AHEAD + 1;
                if (k + ST_AHEAD < RPT)
                    request(r, k + ST_AHEAD, buf[(k + ST_AHEAD) % M], at[(k + ST_AHEAD) % M]);
                const uint4 i = at[k % M];
                const uint32_t all[4] = {i.x, i.y, i.z, i.w};
                uint32_t pair[(W + 1) / 2];
#pragma unroll
                for (int w = 0; w < (W + 1) / 2; ++w)
                    pair[w] = all[w];
                f(k, sum(pair, v, [&](int w) { return buf[k % M][w]; }));
            }
        } else {
#pragma unroll
            for (int k = 0; k < RPT; ++k) {
                uint32_t pair[(W + 1) / 2];
#pragma unroll
                for (int w = 0; w < (W + 1) / 2; ++w) {
                    pair[w] = id[k][w];
                    if constexpr (RPT >= 4)
                        asm volatile("" : "+v"(pair[w]));  // see own_row
                }
                f(k, sum(pair, v, [&](int w) {
                      return w < WR ? a[k][w < WR ? w : 0]
                                    : far[(w - WR) * rows + min(own_row<T, RPT>(k), rows - 1)];
                  }));
            }
        }
    }
};

extern __shared__ double res_lds[];

// What the solvers share: the workgroup's place, its ghosts and its matrix.
// LDS: the vector the next product gathers (own rows, then ghosts), the
// solver's own ghost vectors, the matrix values that are not in registers.
template <int T, int RPT, int W>
struct Res {
    static constexpr bool BIG = RPT >= 8;
    const ResArgs &a;
    ResShared &sh;
    int tid, g, n, R, ng, par;
    const int32_t *gl;
    double *gv;
    double *hist, *scal;
    uint32_t tag, pub;
    GhostWords gw;
    ResRows<T, RPT, W> M;

    // ghost_vectors: how many the solver keeps behind gv
    __device__ __forceinline__ Res(const ResArgs &a_, ResShared &sh_, int ghost_vectors) : a(a_), sh(sh_)
    {
        tid = threadIdx.x;
        g = blockIdx.x;
        n = a.A.n;
        R = a.rows;
        ng = a.gcount[g];
        gv = res_lds;
        // (the last workgroup records: workgroup 0 has the sums to collect)
        hist = g == (int)gridDim.x - 1 ? a.hist : nullptr;
        scal = hist ? a.scal : nullptr;
        par = a.st->it & 1;  // the buffers a resumed solve left r, p, A p in
        tag = a.epoch;
        gw = GhostWords{};
        if (tid == 0) {
            sh.s = *a.st;
            sh.fault = 0;
        }
        M.zero = R + (1 + ghost_vectors) * ng;
        M.far = res_lds + M.zero + 1;
        M.rows = R;
        gl = a.glist + (size_t)g * a.gcap;
        if (tid == 0)
            gv[M.zero] = 0.0;
        M.load(a);
        pub = 0;
#pragma unroll
        for (int k = 0; k < RPT; ++k)
            if (mine(k) && row(k) < n && a.pub[row(k)])
                pub |= 1u << k;
    }

    // (the slice, like own_row's thread, opaque: no condition held per row)
    __device__ __forceinline__ int slice(int k) const
    {
        int s = M.sl[k];
        if constexpr (RPT >= 4)
            asm volatile("" : "+s"(s));
        return s;
    }
    __device__ __forceinline__ bool mine(int k) const { return slice(k) >= 0; }
    __device__ __forceinline__ int row(int k) const { return slice(k) * SLICE + (own_row<T, RPT>(0) & 63); }
    // a uniform base and a 32-bit offset: no 64-bit address per row to hold
    __device__ __forceinline__ static double *at(double *v, int i)
    {
        return reinterpret_cast<double *>(reinterpret_cast<char *>(v) + (uint32_t)i * 8u);
    }
    __device__ __forceinline__ double get(double *v, int k) const
    {
        const int i = row(k);
        return mine(k) && i < n ? *at(v, i) : 0.0;
    }
    __device__ __forceinline__ void put(double *v, int k, double x) const
    {
        const int i = row(k);
        if (mine(k) && i < n)
            *at(v, i) = x;
    }
    // the gathered vector's entry of row k
    __device__ __forceinline__ double own(int k) const
    {
        return mine(k) ? gv[own_row<T, RPT>(k)] : 0.0;
    }
    __device__ __forceinline__ void set_own(int k, double v) const
    {
        if (mine(k))
            gv[own_row<T, RPT>(k)] = v;
    }
    __device__ __forceinline__ const uint64_t *ll() const { return a.ll + (size_t)(tag & 1u) * 2 * (size_t)n; }
    __device__ __forceinline__ void publish(int k, double v) const
    {
        uint32_t bits = pub;
        if constexpr (RPT >= 4)
            asm volatile("" : "+v"(bits));
        if (bits >> k & 1u)
            store_tagged(reinterpret_cast<uint64_t *>(
                             reinterpret_cast<char *>(a.ll + 2 * (size_t)(tag & 1u) * (size_t)n) +
                             (uint32_t)row(k) * 16u),
                         tag, v);
    }
    // f(j, value of the current tag) for every ghost j of this thread
    template <typename F>
    __device__ __forceinline__ void each_ghost(F &&f)
    {
        for (int j0 = 0; j0 < ng; j0 += GPT * T) {
            if (j0 > 0 && !ghost_poll<T>(ll(), gl, ng, tag, gw, j0)) {
                sh.fault = 1;
                return;
            }
#pragma unroll
            for (int i = 0; i < GPT; ++i)
                if (j0 + tid + i * T < ng)
                    f(j0 + tid + i * T, untag(gw.lo[i], gw.hi[i]));
            if (j0 + GPT * T < ng)
                ghost_load<T>(ll(), gl, ng, gw, j0 + GPT * T);
        }
    }
    template <int K, typename FIN>
    __device__ __forceinline__ bool reduce(dd (&v)[K], FIN &&fin)
    {
        if (all_reduce<T, K, BIG ? 2 : 4>(v, sh, a, g, tag, ll(), gl, ng, gw, fin))
            return true;
        a.ctl->fault = a.epoch;
        return false;
    }
    __device__ __forceinline__ bool start()
    {
        if (everyone_here<T>(sh, a, g))
            return true;
        if (tid == 0)
            a.ctl->declined = a.epoch;
        return false;
    }
    // f(k, row k of the product with gv), the row published.
    template <typename F>
    __device__ __forceinline__ void product(F &&f) const
    {
        M.product(a, gv, [&](int k, double q) {
            publish(k, q);
            f(k, q);
        });
    }
    // Entries of N rows from k0 of a vector kept in memory, requested together
    // (a load after the store of another row would wait for its own trip).
    template <int N>
    __device__ __forceinline__ void get_rows(double *v, int k0, double (&out)[N]) const
    {
#pragma unroll
        for (int k = 0; k < N; ++k)
            out[k] = get(v, k0 + k);
    }
    // r_0 = b - A x_0 into r, published; its reduction (FIN_SETUP).
    __device__ __forceinline__ bool residual(double (&r)[RPT])
    {
#pragma unroll
        for (int k = 0; k < RPT; ++k)
            set_own(k, get(a.x, k));
        for (int j = tid; j < ng; j += T)
            gv[R + j] = a.x[gl[j]];
        __syncthreads();
        dd acc[2] = {dd{0.0, 0.0}, dd{0.0, 0.0}};
        M.product(a, gv, [&](int k, double q) {
            const double bi = get(const_cast<double *>(a.b), k);
            const double ri = bi - q;
            r[k] = ri;
            publish(k, ri);
            dd_fma(acc[0], ri, ri);
            dd_fma(acc[1], bi, bi);
        });
        return reduce(acc, [&](const double *d) {
            if (tid == 0)
                finalize(&sh.s, FIN_SETUP, d, 2, hist, scal);
        });
    }
};

// Above this sqrt(v) > tol for certain (v the square of a norm), so the
// test against the tolerance needs the square root only near its end.
__device__ __forceinline__ double near_of(double tol)
{
    return tol > 1e-150 ? tol * tol * (1.0 + 1e-12) : HUGE_VAL;
}

// The scalars of the loops below: wave 0 of every workgroup computes them from
// registers, with finalize's expressions, and leaves what the other waves
// need in LDS; the residual norm's quotient only feeds the history, so it
// stays off the path between two products.

// ---------------------------------------------------------------------- CG

struct CgScalars {
    double bnorm, tol, near, alpha, beta, rr;
    int max_iter, it0, it, status;

    __device__ __forceinline__ explicit CgScalars(const DevState &s)
        : bnorm(s.bnorm), tol(s.tol), near(near_of(s.tol)), alpha(s.alpha), beta(s.beta), rr(s.rr),
          max_iter(s.max_iter), it0(s.it), it(s.it), status(s.status)
    {
    }
    // FIN_CG_RR_ALPHA on d = {<p,Ap>, <Ap,Ap>, <r,r>}, by wave 0
    __device__ __forceinline__ void step(const double *d, ResShared &sh) const
    {
        const double rr1 = d[2];
        int st = ST_RUNNING;
        double al = alpha, be = beta;
        if (!isfinite(rr1))
            st = ST_BREAKDOWN;
        else if (rr1 <= near && sqrt(rr1) <= tol)
            st = ST_CONVERGED;
        else if (it + 1 >= max_iter)
            st = ST_NOT_CONVERGED;
        else if (!(d[0] > 0.0) || !isfinite(d[0]) || !isfinite(d[1]))
            st = ST_BREAKDOWN;
        else {
            al = rr1 / d[0];
            be = al * al * d[1] / rr1 - 1.0;  // Eq. (3)
        }
        if (threadIdx.x == 0) {
            sh.alpha = al;
            sh.beta = be;
            sh.status = st;
            sh.s.rr = rr1;
        }
    }
    // by every thread, after the reduction; records where hist is set
    __device__ __forceinline__ void take(const ResShared &sh, double *hist, double *scal)
    {
        ++it;
        alpha = sh.alpha;
        beta = sh.beta;
        status = sh.status;
        rr = sh.s.rr;
        if (threadIdx.x == 0 && hist) {
            put_hist(&sh.s, hist, it, sqrt(rr) / bnorm);
            put_scal(&sh.s, scal, it - 1, 3, rr);
            if (status == ST_RUNNING) {
                put_scal(&sh.s, scal, it, 0, alpha);
                put_scal(&sh.s, scal, it, 1, beta);
            }
        }
    }
    // the solver state, by one thread
    __device__ __forceinline__ void leave(DevState &s, DevState *out) const
    {
        if (it > it0) {
            s.it = it;
            s.status = status;
            s.alpha = alpha;
            s.beta = beta;
            s.last_rel = sqrt(rr) / bnorm;
        }
        *out = s;
    }
};

template <int T, int RPT, int W>
__global__ __launch_bounds__(T) void k_res_cg(ResArgs a)
{
    __shared__ ResShared sh;
    Res<T, RPT, W> c(a, sh, 1);
    constexpr bool BIG = Res<T, RPT, W>::BIG;   // p only in LDS
    double *rg = c.gv + c.R + c.ng;            // r of the ghosts
    double *pg = c.gv + c.R;                   // p of the ghosts
    double xr[RPT], rr[RPT], ap[RPT];
    [[maybe_unused]] double pr[BIG ? 1 : RPT];
#pragma unroll
    for (int k = 0; k < RPT; ++k) {
        rr[k] = a.resume ? c.get(a.r[c.par], k) : 0.0;
        ap[k] = a.resume ? c.get(a.ap[c.par], k) : 0.0;
        xr[k] = c.get(a.x, k);
    }
    if (!c.start())
        return;
    auto p_of = [&](int k) {
        if constexpr (BIG)
            return c.own(k);
        else
            return pr[k];
    };
    auto p_set = [&](int k, double v) {
        if constexpr (!BIG)
            pr[k] = v;
        c.set_own(k, v);
    };
    auto product = [&](dd &pap, dd &apap) {
        c.product([&](int k, double q) {
            ap[k] = q;
            dd_fma(pap, q, p_of(k));
            dd_fma(apap, q, q);
            settle<BIG>(pap);
            settle<BIG>(apap);
        });
    };
    if (!a.resume) {
        if (!c.residual(rr))
            return;
        if (sh.s.status == ST_RUNNING) {
#pragma unroll
            for (int k = 0; k < RPT; ++k)
                p_set(k, rr[k]);
            c.each_ghost([&](int j, double v) { rg[j] = pg[j] = v; });
            __syncthreads();
            ++c.tag;
            dd acc[2] = {dd{0.0, 0.0}, dd{0.0, 0.0}};
            product(acc[0], acc[1]);
            if (!c.reduce(acc, [&](const double *d) {
                    if (c.tid == 0)
                        finalize(&sh.s, FIN_CG_ALPHA, d, 2, c.hist, c.scal);
                }))
                return;
        }
    } else {
        // r, p of the ghosts from where their owners left them; A p again by words
#pragma unroll
        for (int k = 0; k < RPT; ++k) {
            c.publish(k, ap[k]);
            p_set(k, c.get(a.p[c.par], k));
        }
        for (int j = c.tid; j < c.ng; j += T) {
            rg[j] = a.r[c.par][c.gl[j]];
            pg[j] = a.p[c.par][c.gl[j]];
        }
        ghost_load<T>(c.ll(), c.gl, c.ng, c.gw);
        if (!ghost_poll<T>(c.ll(), c.gl, c.ng, c.tag, c.gw))
            sh.fault = 1;
        __syncthreads();
    }
    CgScalars z(sh.s);
    while (z.status == ST_RUNNING && z.it - z.it0 < a.chunk) {
        const double alpha = z.alpha, beta = z.beta;
        dd acc[3] = {dd{0.0, 0.0}, dd{0.0, 0.0}, dd{0.0, 0.0}};
        // x_i, r_i, p_i and <r_i, r_i>; r_i, p_i of the ghosts
        c.each_ghost([&](int j, double v) {
            const double ri = rg[j] - alpha * v;
            rg[j] = ri;
            pg[j] = ri + beta * pg[j];
        });
#pragma unroll
        for (int k = 0; k < RPT; ++k) {
            const double pi = p_of(k);
            xr[k] = xr[k] + alpha * pi;
            const double ri = rr[k] - alpha * ap[k];
            rr[k] = ri;
            p_set(k, ri + beta * pi);
            dd_fma(acc[2], ri, ri);
        }
        settle<BIG>(acc[2]);
        __syncthreads();
        ++c.tag;
        product(acc[0], acc[1]);
        if (!c.reduce(acc, [&](const double *d) { z.step(d, sh); }))
            return;
        z.take(sh, c.hist, c.scal);
    }
    const bool more = z.status == ST_RUNNING;  // the chunk ended first
    const int end = z.it & 1;
#pragma unroll
    for (int k = 0; k < RPT; ++k) {
        c.put(a.x, k, xr[k]);
        if (more) {
            c.put(a.r[end], k, rr[k]);
            c.put(a.p[end], k, p_of(k));
            c.put(a.ap[end], k, ap[k]);
        }
    }
    if (c.g == 0 && c.tid == 0)
        z.leave(sh.s, a.st);
}

// ---------------------------------------------------------------- BiCGStab

// Algorithm 4 with the two reduction points of the two-kernel schedule: A p
// with {<Ap,r0*>, <r,r0*>, <r,r>}, then A s with {<As,s>, <As,As>, <As,r0*>,
// <s,s>}.  A ghost's r and A p share a slot (A p replaces r when s is
// formed, r the A p when p is); p has one of its own, the gathered vector
// being s meanwhile.
template <int T, int RPT, int W>
__global__ __launch_bounds__(T) void k_res_bicg(ResArgs a)
{
    __shared__ ResShared sh;
    Res<T, RPT, W> c(a, sh, 2);
    constexpr bool BIG = Res<T, RPT, W>::BIG;  // x and r0* in memory (the XCD's L2)
    double *sg = c.gv + c.R, *pg = sg + c.ng, *rg = pg + c.ng;
    double rr[RPT], pr[RPT], ap[RPT], as[RPT];
    [[maybe_unused]] double xr[BIG ? 1 : RPT], rs[BIG ? 1 : RPT];
#pragma unroll
    for (int k = 0; k < RPT; ++k) {
        as[k] = 0.0;
        rr[k] = a.resume ? c.get(a.r[c.par], k) : 0.0;
        pr[k] = a.resume ? c.get(a.p[c.par], k) : 0.0;
        ap[k] = a.resume ? c.get(a.ap[c.par], k) : 0.0;
        if constexpr (!BIG) {
            xr[k] = c.get(a.x, k);
            rs[k] = a.resume ? c.get(a.rs, k) : 0.0;
        }
    }
    if (!c.start())
        return;
    double mem[RPT];  // r0* or x of the rows, from memory for one phase
    auto rs_of = [&](int k) {
        if constexpr (BIG)
            return mem[k];
        else
            return rs[k];
    };
    double alpha = 0.0, rho = 0.0;
    // A p (gathered) and the reduction point after it; dots[1], dots[2] come in
    auto ap_step = [&](dd (&acc)[3], bool first) -> bool {
        if constexpr (BIG)
            c.get_rows(a.rs, 0, mem);
        __syncthreads();
        ++c.tag;
        c.product([&](int k, double q) {
            ap[k] = q;
            dd_fma(acc[0], q, rs_of(k));
            settle<BIG>(acc[0]);
        });
        const double rho0 = rho;
        if (!c.reduce(acc, [&](const double *d) {  // FIN_B_RHO_ALPHA / FIN_B_XRP_ALPHA
                const double apr = d[0], rh = first ? rho0 : d[1];
                const bool bad = apr == 0.0 || !isfinite(apr) || rh == 0.0 || !isfinite(rh);
                if (c.tid == 0) {
                    sh.s.rho = rh;
                    if (!first)
                        sh.s.rr = d[2];
                    if (!bad)
                        sh.s.apr = apr;
                    sh.alpha = bad ? alpha : rh / apr;
                    sh.status = bad ? ST_BREAKDOWN : ST_RUNNING;
                }
            }))
            return false;
        alpha = sh.alpha;
        rho = sh.s.rho;
        return true;
    };
    int status;
    if (!a.resume) {
        if (!c.residual(rr))
            return;
#pragma unroll
        for (int k = 0; k < RPT; ++k) {
            pr[k] = rr[k];
            c.put(a.rs, k, rr[k]);  // r0* = r0 (a resumed solve reads it back)
            if constexpr (!BIG)
                rs[k] = rr[k];
        }
        status = sh.s.status;
        if (status == ST_RUNNING) {
            rho = sh.s.rho;
#pragma unroll
            for (int k = 0; k < RPT; ++k)
                c.set_own(k, rr[k]);
            c.each_ghost([&](int j, double v) { sg[j] = pg[j] = rg[j] = v; });
            dd acc[3] = {dd{0.0, 0.0}, dd{0.0, 0.0}, dd{0.0, 0.0}};
            if (!ap_step(acc, true))
                return;
            status = sh.status;
            if (c.tid == 0 && status == ST_RUNNING)
                put_scal(&sh.s, c.scal, 0, 0, alpha);
        }
    } else {
#pragma unroll
        for (int k = 0; k < RPT; ++k)
            c.publish(k, ap[k]);
        for (int j = c.tid; j < c.ng; j += T) {
            rg[j] = a.r[c.par][c.gl[j]];
            pg[j] = a.p[c.par][c.gl[j]];
        }
        ghost_load<T>(c.ll(), c.gl, c.ng, c.gw);
        if (!ghost_poll<T>(c.ll(), c.gl, c.ng, c.tag, c.gw))
            sh.fault = 1;
        __syncthreads();
        alpha = sh.s.alpha;
        rho = sh.s.rho;
        status = sh.s.status;
    }
    const double bnorm = sh.s.bnorm, tol = sh.s.tol, near = near_of(tol);
    const int max_iter = sh.s.max_iter, it0 = sh.s.it;
    int it = it0;
    double rr_next = 0.0;
    while (status == ST_RUNNING && it - it0 < a.chunk) {
        // s = r - alpha A p, A s and its inner products
        c.each_ghost([&](int j, double v) {
            sg[j] = rg[j] - alpha * v;
            rg[j] = v;
        });
        dd acc[4] = {dd{0.0, 0.0}, dd{0.0, 0.0}, dd{0.0, 0.0}, dd{0.0, 0.0}};
#pragma unroll
        for (int k = 0; k < RPT; ++k) {
            const double si = rr[k] - alpha * ap[k];
            c.set_own(k, si);
            dd_fma(acc[3], si, si);
        }
        settle<BIG>(acc[3]);
        if constexpr (BIG)
            c.get_rows(a.rs, 0, mem);
        __syncthreads();
        ++c.tag;
        c.product([&](int k, double q) {
            as[k] = q;
            dd_fma(acc[0], q, c.own(k));
            dd_fma(acc[1], q, q);
            dd_fma(acc[2], q, rs_of(k));
            settle<BIG>(acc[0]);
            settle<BIG>(acc[1]);
            settle<BIG>(acc[2]);
        });
        if (!c.reduce(acc, [&](const double *d) {  // FIN_B_SS_OMEGA
                const double ass = d[0], asas = d[1], asr = d[2], ss = d[3];
                int st = ST_RUNNING;
                double be = 0.0, om = 0.0, rn = 0.0;
                if (ss <= near && sqrt(ss) <= tol)
                    st = ST_HALF;
                else if (asas == 0.0 || !isfinite(asas) || !isfinite(ass) || !isfinite(asr))
                    st = ST_BREAKDOWN;
                else {
                    be = -asr / sh.s.apr;  // via <s_i, r0*> = 0
                    om = ass / asas;
                    rn = ss - 2.0 * om * ass + om * om * asas;
                    if (!isfinite(rn))
                        st = ST_FINAL_BREAKDOWN;
                    else if (rn <= near && sqrt(rn > 0.0 ? rn : 0.0) <= tol)
                        st = ST_FINAL_CONVERGED;
                    else if (om == 0.0)
                        st = ST_FINAL_BREAKDOWN;
                    else if (it + 1 >= max_iter)
                        st = ST_FINAL_NOT_CONVERGED;
                }
                if (c.tid == 0) {
                    sh.s.ss = ss;
                    sh.beta = be;
                    sh.omega = om;
                    sh.rr_next = rn;
                    sh.status = st;
                }
            }))
            return;
        status = sh.status;
        if (status == ST_BREAKDOWN)
            break;
        const double beta = sh.beta, omega = sh.omega;
        rr_next = status == ST_HALF ? sh.s.ss : sh.rr_next;
        if (status == ST_HALF) {
            if constexpr (BIG)
                c.get_rows(a.x, 0, mem);
#pragma unroll
            for (int k = 0; k < RPT; ++k) {
                if constexpr (BIG)
                    c.put(a.x, k, mem[k] + alpha * pr[k]);
                else
                    xr[k] = xr[k] + alpha * pr[k];
            }
            ++it;
            break;
        }
        // x, r, p of the next iteration; r, p of the ghosts
        c.each_ghost([&](int j, double v) {
            const double ri = sg[j] - omega * v;
            const double pn = ri + beta * (pg[j] - omega * rg[j]);
            rg[j] = ri;
            pg[j] = sg[j] = pn;
        });
        dd acc3[3] = {dd{0.0, 0.0}, dd{0.0, 0.0}, dd{0.0, 0.0}};
        if constexpr (BIG) {
            c.get_rows(a.x, 0, mem);
#pragma unroll
            for (int k = 0; k < RPT; ++k)
                mem[k] = mem[k] + alpha * pr[k] + omega * c.own(k);
#pragma unroll
            for (int k = 0; k < RPT; ++k)
                c.put(a.x, k, mem[k]);
            c.get_rows(a.rs, 0, mem);
        }
#pragma unroll
        for (int k = 0; k < RPT; ++k) {
            const double si = c.own(k), pi = pr[k];
            if constexpr (!BIG)
                xr[k] = xr[k] + alpha * pi + omega * si;
            const double ri = si - omega * as[k];
            rr[k] = ri;
            const double pn = ri + beta * (pi - omega * ap[k]);
            pr[k] = pn;
            c.set_own(k, pn);
            dd_fma(acc3[1], ri, rs_of(k));
            dd_fma(acc3[2], ri, ri);
        }
        settle<BIG>(acc3[1]);
        settle<BIG>(acc3[2]);
        ++it;
        if (c.tid == 0 && c.hist) {
            put_hist(&sh.s, c.hist, it, sqrt(rr_next > 0.0 ? rr_next : 0.0) / bnorm);
            put_scal(&sh.s, c.scal, it - 1, 1, beta);
            put_scal(&sh.s, c.scal, it - 1, 2, omega);
            put_scal(&sh.s, c.scal, it - 1, 3, rr_next);
        }
        if (status != ST_RUNNING) {  // decided: only the last <r,r0*>, <r,r> are left
            ++c.tag;
            __syncthreads();
#pragma unroll
            for (int k = 0; k < RPT; ++k)
                c.publish(k, rr[k]);  // (every reduction is followed by the ghosts' words)
            if (!c.reduce(acc3, [&](const double *d) {
                    if (c.tid == 0) {
                        sh.s.rho = d[1];
                        sh.s.rr = d[2];
                    }
                }))
                return;
            break;
        }
        if (!ap_step(acc3, false))
            return;
        status = sh.status;
        if (c.tid == 0 && status == ST_RUNNING)
            put_scal(&sh.s, c.scal, it, 0, alpha);
    }
    const bool more = status == ST_RUNNING;  // the chunk ended first
    const int end = it & 1;
#pragma unroll
    for (int k = 0; k < RPT; ++k) {
        if constexpr (!BIG)
            c.put(a.x, k, xr[k]);
        if (more) {
            c.put(a.r[end], k, rr[k]);
            c.put(a.p[end], k, pr[k]);
            c.put(a.ap[end], k, ap[k]);
        }
    }
    if (c.tid == 0 && c.hist && status == ST_HALF) {
        put_hist(&sh.s, c.hist, it, sqrt(rr_next) / bnorm);
        put_scal(&sh.s, c.scal, it - 1, 3, rr_next);
    }
    if (c.g == 0 && c.tid == 0) {
        sh.s.alpha = alpha;
        sh.s.rho_pub = 0;
        if (it > it0) {
            sh.s.it = it;
            sh.s.beta = sh.beta;
            sh.s.omega = sh.omega;
            sh.s.rr_next = sh.rr_next;
            sh.s.last_rel = sqrt(rr_next > 0.0 ? rr_next : 0.0) / bnorm;
        }
        sh.s.status = status == ST_HALF || status == ST_FINAL_CONVERGED ? ST_CONVERGED
                      : status == ST_FINAL_NOT_CONVERGED                ? ST_NOT_CONVERGED
                      : status == ST_FINAL_BREAKDOWN                    ? ST_BREAKDOWN
                                                                        : status;
        *a.st = sh.s;
    }
}

}  // namespace

// ------------------------------------------------------------------ host

namespace {

// Static LDS of the kernels (ResShared) and a margin.
constexpr size_t RES_STATIC_LDS = sizeof(ResShared) + 512;

using ResKernel = void (*)(ResArgs);

// Threads and rows per thread: the fewest waves whose threads keep at most
// eight rows, since every wave joins each reduction.  Kernels for at most
// five and at most seven entries per row.
struct ResBody {
    int threads, rpt;
    ResKernel cg[2], bicg[2];
};
#define RES_BODY(T, RPT)                                                                        \
    {                                                                                           \
        T, RPT, {k_res_cg<T, RPT, 5>, k_res_cg<T, RPT, 7>}, { k_res_bicg<T, RPT, 5>, k_res_bicg<T, RPT, 7> } \
    }
const ResBody BODIES[] = {RES_BODY(256, 1), RES_BODY(256, 2), RES_BODY(512, 2), RES_BODY(512, 4), RES_BODY(512, 8),
                          {512, 16, {k_res_cg<512, 16, 5>, k_res_cg<512, 16, 7>}, {nullptr, nullptr}}};
#undef RES_BODY

int width_class(const DevCsr &A) { return A.max_width <= 5 ? 0 : 1; }

// Doubles of dynamic LDS: the gathered vector, the ghost vectors, the
// matrix values that are not in registers.
size_t res_lds_doubles(const ResShape &sh, const DevCsr &A, int ghosts)
{
    const int far = res_lds_values(BODIES[sh.body].rpt, width_class(A) ? 7 : 5);
    return (size_t)sh.rows * (1 + far) + (size_t)(sh.bicg ? 3 : 2) * ghosts + 1;
}

}  // namespace

bool resident_shape(const DevCsr &A, bool bicg, int units, size_t max_lds, int first, ResShape *out)
{
    if (A.nslices <= 0 || A.max_width < 1 || A.max_width > 7 || units < 1)
        return false;
    const int gmax = units < RES_MAX_WG ? units : RES_MAX_WG;
    int64_t rows = ((int64_t)A.nslices + gmax - 1) / gmax * SLICE;
    if (gmax > 1 && rows < 256)
        rows = 256;
    for (int i = first; i < (int)(sizeof(BODIES) / sizeof(BODIES[0])); ++i) {
        if ((int64_t)BODIES[i].threads * BODIES[i].rpt < rows)
            continue;
        if (bicg && !BODIES[i].bicg[0])
            return false;
        ResShape sh;
        sh.body = i;
        sh.bicg = bicg;
        sh.rows = (int)rows;
        sh.groups = (int)(((int64_t)A.n + rows - 1) / rows);
        const size_t lds = res_lds_doubles(sh, A, 0) * 8 + RES_STATIC_LDS;
        if (lds > max_lds || sh.groups > RES_MAX_WG)
            return false;
        const int64_t gcap = (int64_t)((max_lds - lds) / (bicg ? 24 : 16));
        sh.gcap = (int)(gcap < 65534 - rows ? gcap : 65534 - rows);
        *out = sh;
        return true;
    }
    return false;
}

hipError_t launch_res_plan(const DevCsr &A, const ResShape &sh, const int32_t *perm, const int32_t *owner,
                           uint16_t *idx, int32_t *gcount, int32_t *glist, uint8_t *pub, hipStream_t s)
{
    hipLaunchKernelGGL(k_res_plan, dim3(sh.groups), dim3(PLAN_T), 0, s, A, sh.rows / SLICE, sh.gcap, perm, owner, idx,
                       gcount, glist, pub);
    return hipGetLastError();
}

bool resident_streams(const ResShape &sh) { return res_streamed(BODIES[sh.body].rpt); }

hipError_t launch_res_pack(const DevCsr &A, const ResShape &sh, const int32_t *owner, const int32_t *gcount,
                           const uint16_t *idx, uint4 *out, hipStream_t s)
{
    hipLaunchKernelGGL(k_res_pack, dim3((A.nslices + 3) / 4), dim3(256), 0, s, A, sh.rows, owner, gcount, idx, out);
    return hipGetLastError();
}

hipError_t launch_resident(const ResShape &sh, const ResArgs &a, hipStream_t s)
{
    const int w = width_class(a.A);
    const ResBody &b = BODIES[sh.body];
    hipLaunchKernelGGL(sh.bicg ? b.bicg[w] : b.cg[w], dim3(sh.groups), dim3(b.threads),
                       (uint32_t)(res_lds_doubles(sh, a.A, sh.ghosts) * 8), s, a);
    return hipGetLastError();
}

}  // namespace fk
