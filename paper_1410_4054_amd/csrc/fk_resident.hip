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
__global__ __launch_bounds__(PLAN_T) void k_res_plan(DevCsr A, int rows, int gcap, uint16_t *idx, int32_t *gcount,
                                                     int32_t *glist, uint8_t *pub)
{
    __shared__ uint32_t bits[RES_PLAN_WORDS];
    __shared__ uint32_t pre[PLAN_T];
    __shared__ int lo_s, hi_s;
    const int g = blockIdx.x, tid = threadIdx.x, lane = tid & 63;
    const int row0 = g * rows, row1 = min(A.n, row0 + rows);
    const int s0 = row0 / SLICE, s1 = (row1 + SLICE - 1) / SLICE;
    if (tid == 0) {
        lo_s = row0;
        hi_s = row1 - 1;
    }
    __syncthreads();
    int lo = row0, hi = row1 - 1;
    for (int sl = s0 + tid / 64; sl < s1; sl += PLAN_T / 64) {
        const int e0 = A.sell_ptr[sl], width = (A.sell_ptr[sl + 1] - e0) / SLICE, row = sl * SLICE + lane;
        for (int k = 0; k < width; ++k) {
            const int c = row < A.n ? entry_col(A, sl, e0, k, lane, row) : -1;
            if (c >= 0) {
                lo = min(lo, c);
                hi = max(hi, c);
            }
        }
    }
    atomicMin(&lo_s, lo);
    atomicMax(&hi_s, hi);
    __syncthreads();
    lo = lo_s;
    const int64_t span = (int64_t)hi_s - lo + 1;
    if (span > (int64_t)RES_PLAN_WORDS * 32) {
        if (tid == 0)
            gcount[g] = -1;
        return;
    }
    const int nw = (int)((span + 31) / 32);
    for (int w = tid; w < nw; w += PLAN_T)
        bits[w] = 0;
    __syncthreads();
    for (int sl = s0 + tid / 64; sl < s1; sl += PLAN_T / 64) {
        const int e0 = A.sell_ptr[sl], width = (A.sell_ptr[sl + 1] - e0) / SLICE, row = sl * SLICE + lane;
        for (int k = 0; k < width; ++k) {
            const int c = row < A.n ? entry_col(A, sl, e0, k, lane, row) : -1;
            if (c >= 0 && (c < row0 || c >= row1))
                atomicOr(&bits[(c - lo) >> 5], 1u << ((c - lo) & 31));
        }
    }
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
    for (int sl = s0 + tid / 64; sl < s1; sl += PLAN_T / 64) {
        const int e0 = A.sell_ptr[sl], width = (A.sell_ptr[sl + 1] - e0) / SLICE, row = sl * SLICE + lane;
        for (int k = 0; k < width; ++k) {
            const int c = row < A.n ? entry_col(A, sl, e0, k, lane, row) : -1;
            uint32_t v = RES_NONE;
            if (c >= row0 && c < row1) {
                v = (uint32_t)(c - row0);
            } else if (c >= 0) {
                const int w = (c - lo) >> 5, t = w / per;
                uint32_t r = t > 0 ? pre[t - 1] : 0;
                for (int u = t * per; u < w; ++u)
                    r += __popc(bits[u]);
                r += __popc(bits[w] & ((1u << ((c - lo) & 31)) - 1u));
                v = (uint32_t)rows + r;
            }
            idx[e0 + k * SLICE + lane] = (uint16_t)v;
        }
    }
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

struct ResShared {
    DevState s;
    dd rows[32][4];  // per row of 16 lanes of each wave: the four dots
    dd psum[RES_MAX_WG / 64][4];
    double alpha, beta;
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

template <int T>
__device__ __forceinline__ void ghost_load(const uint64_t *ll, const int32_t *gl, int ng, GhostWords &w, int j0 = 0)
{
#pragma unroll
    for (int i = 0; i < GPT; ++i) {
        const int j = j0 + (int)threadIdx.x + i * T;
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
// (2D Poisson 255^2, 255 workgroups: 8.9 us per iteration).  Waves that
// collect nothing poll the thread's ghost words meanwhile.  Returns false
// when a wait ran out; ends past a barrier.
template <int T, int K, typename FIN>
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
        if (lane < K) {
            store_tagged(part + (size_t)16 * g + 4 * lane, tag, r.hi);
            store_tagged(part + (size_t)16 * g + 4 * lane + 2, tag, r.lo);
        }
    }
    dd mine{0.0, 0.0};
    if (wave < np) {
        // lane: dot l & 3 of the members (l >> 2) + 16 i of the wave's 64
        const int m = wave * 64 + (lane >> 2);
        uint64_t w[16] = {};
        bool ok = dot >= K;
        for (int spin = 0;; ++spin) {
            if (!ok) {
                ok = true;
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    if (m + 16 * i < G) {
#pragma unroll
                        for (int j = 0; j < 4; ++j)
                            w[4 * i + j] = load_word(part + (size_t)16 * (m + 16 * i) + 4 * dot + j);
                    }
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    if (m + 16 * i < G)
                        ok = ok && tagged(w[4 * i], w[4 * i + 1], tag) && tagged(w[4 * i + 2], w[4 * i + 3], tag);
            }
            if (__builtin_amdgcn_ballot_w64(!ok) == 0)
                break;
            if (spin >= FK_RES_SPIN_LIMIT) {
                sh.fault = 1;
                break;
            }
        }
        dd q[4];  // members past G and dots past K: words of zero, sums of zero
#pragma unroll
        for (int i = 0; i < 4; ++i)
            q[i] = dd{untag(w[4 * i], w[4 * i + 1]), untag(w[4 * i + 2], w[4 * i + 3])};
        ghost_load<T>(ll, gl, ng, gw);  // in flight during the sums; checked after the last barrier
        mine = wave_quads(dd_add(dd_add(q[0], q[1]), dd_add(q[2], q[3])));
        if (np > 1 && lane < 4)
            sh.psum[wave][dot] = mine;
    } else if (wave > 0) {
        if (!ghost_poll<T>(ll, gl, ng, tag, gw))
            sh.fault = 1;
    } else {
        ghost_load<T>(ll, gl, ng, gw);
    }
    if (np > 1)
        __syncthreads();
    if (wave == 0) {
        double d[K];
        if (np > 0) {
            for (int w = 1; w < np; ++w)
                mine = dd_add(mine, sh.psum[w][dot]);
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

// Index of the thread's row k among the workgroup's.  With eight rows per
// thread the compiler must not compute what follows from it (addresses,
// bounds, unpacked indices of every row) once and hold it over the whole
// solve: that spills the 256 registers.
template <int T, int RPT>
__device__ __forceinline__ int own_row(int k)
{
    int t = threadIdx.x;
    if constexpr (RPT >= 8)
        asm volatile("" : "+v"(t));
    return k * T + t;
}

// Values of a row held in LDS instead of registers: two of five with eight
// rows per thread, whose 256 registers do not hold all of them (all in
// registers: 202 spilled, 1000^2 Poisson 21 us per iteration).
constexpr int res_lds_values(int rpt) { return rpt >= 8 ? 2 : 0; }

// The workgroup's rows of the matrix: row k of thread t is k T + t, so a
// wave holds whole slices.
template <int T, int RPT, int W>
struct ResRows {
    static constexpr int WL = res_lds_values(RPT), WR = W - WL;
    double a[RPT][WR];
    double *far;  // values WR .. W-1 of the workgroup's rows, [WL][rows]
    int rows;
    uint32_t id[RPT][(W + 1) / 2];  // two 16-bit indices to a word

    __device__ __forceinline__ void load(const ResArgs &r, int row0)
    {
        const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x / SLICE)), lane = threadIdx.x & 63;
#pragma unroll
        for (int k = 0; k < RPT; ++k) {
            const int off = k * T + wave * SLICE;
            const int sl = (row0 + off) / SLICE;
            int e0 = 0, width = 0;
            if (off < r.rows && sl < r.A.nslices) {
                e0 = __builtin_amdgcn_readfirstlane(r.A.sell_ptr[sl]);
                width = (__builtin_amdgcn_readfirstlane(r.A.sell_ptr[sl + 1]) - e0) / SLICE;
            }
#pragma unroll
            for (int w = 0; w < (W + 1) / 2; ++w)
                id[k][w] = RES_NONE | RES_NONE << 16;
#pragma unroll
            for (int w = 0; w < W; ++w) {
                const double v = w < width ? r.A.sell_vals[e0 + w * SLICE + lane] : 0.0;
                if (w < WR)
                    a[k][w < WR ? w : 0] = v;
                else if (off < r.rows)
                    far[(w - WR) * r.rows + k * T + threadIdx.x] = v;
                if (w < width) {
                    const uint32_t i = r.idx[e0 + w * SLICE + lane];
                    id[k][w / 2] = w & 1 ? (id[k][w / 2] & 0xffffu) | i << 16 : (id[k][w / 2] & 0xffff0000u) | i;
                }
            }
        }
    }

    // Row k times v (own rows, then ghosts), left to right.
    __device__ __forceinline__ double dot(int k, const double *v) const
    {
        double q = 0.0;
        uint32_t pair[(W + 1) / 2];
#pragma unroll
        for (int w = 0; w < (W + 1) / 2; ++w) {
            pair[w] = id[k][w];
            if constexpr (RPT >= 8)
                asm volatile("" : "+v"(pair[w]));  // see own_row
        }
#pragma unroll
        for (int w = 0; w < W; ++w) {
            const uint32_t i = w & 1 ? pair[w / 2] >> 16 : pair[w / 2] & 0xffffu;
            const bool on = i != RES_NONE;
            const double av = w < WR ? a[k][w < WR ? w : 0] : far[(w - WR) * rows + min(own_row<T, RPT>(k), rows - 1)];
            const double t = q + av * v[on ? i : 0];
            q = on ? t : q;
        }
        return q;
    }
};

extern __shared__ double res_lds[];

template <int T, int RPT, int W>
__global__ __launch_bounds__(T) void k_res_cg(ResArgs a)
{
    __shared__ ResShared sh;
    const int tid = threadIdx.x;
    const int g = blockIdx.x;
    const int n = a.A.n, R = a.rows, row0 = g * R;
    const int ng = a.gcount[g];
    const int32_t *gl = a.glist + (size_t)g * a.gcap;
    double *pv = res_lds;          // p (first x0): own rows, then ghosts
    double *rg = res_lds + R + ng;  // r of the ghosts
    // (the last workgroup: workgroup 0 has the sums to collect)
    double *hist = g == (int)gridDim.x - 1 ? a.hist : nullptr, *scal = hist ? a.scal : nullptr;
    const int par = a.st->it & 1;  // the buffers a resumed solve left r, p, A p in
    if (tid == 0) {
        sh.s = *a.st;
        sh.fault = 0;
    }
    ResRows<T, RPT, W> M;
    M.far = rg + ng;
    M.rows = R;
    M.load(a, row0);
    constexpr bool P_LDS = RPT >= 8;
    constexpr bool X_MEM = RPT >= 8;  // x stays in memory (the XCD's L2): read and written once an iteration
    double rr[RPT], ap[RPT];
    [[maybe_unused]] double xr[X_MEM ? 1 : RPT];
    [[maybe_unused]] double pr[P_LDS ? 1 : RPT];
    uint32_t pub = 0;
#pragma unroll
    for (int k = 0; k < RPT; ++k) {
        const int li = k * T + tid, row = row0 + li;
        rr[k] = ap[k] = 0.0;
        if constexpr (!X_MEM)
            xr[k] = li < R && row < n ? a.x[row] : 0.0;
        if (li < R && row < n) {
            if (a.pub[row])
                pub |= 1u << k;
            if (a.resume) {
                rr[k] = a.r[par][row];
                ap[k] = a.ap[par][row];
            }
        }
    }
    if (!everyone_here<T>(sh, a, g)) {
        if (tid == 0)
            a.ctl->declined = a.epoch;
        return;
    }
    uint32_t tag = a.epoch;
    auto ll = [&]() { return a.ll + (size_t)(tag & 1u) * 2 * (size_t)n; };
    GhostWords gw{};
    // every ghost's word of the current tag: f(j, value)
    auto each_ghost = [&](auto &&f) -> bool {
        for (int j0 = 0; j0 < ng; j0 += GPT * T) {
            if (j0 > 0 && !ghost_poll<T>(ll(), gl, ng, tag, gw, j0))
                return false;
#pragma unroll
            for (int i = 0; i < GPT; ++i)
                if (j0 + tid + i * T < ng)
                    f(j0 + tid + i * T, untag(gw.lo[i], gw.hi[i]));
            if (j0 + GPT * T < ng)
                ghost_load<T>(ll(), gl, ng, gw, j0 + GPT * T);
        }
        return true;
    };
    auto publish = [&](int k, double v) {
        // a uniform base and a 32-bit offset: no 64-bit address per row held
        if (pub >> k & 1u)
            store_tagged(reinterpret_cast<uint64_t *>(reinterpret_cast<char *>(ll() + 2 * (size_t)row0) +
                                                      (uint32_t)own_row<T, RPT>(k) * 16u),
                         tag, v);
    };
    // p of row k: beside the matrix in a register, or (eight rows) where the
    // gathers read it
    auto p_of = [&](int k) {
        if constexpr (P_LDS) {
            const int li = own_row<T, RPT>(k);
            return li < R ? pv[li] : 0.0;
        } else {
            return pr[k];
        }
    };
    auto p_set = [&](int k, double v) {
        if constexpr (!P_LDS)
            pr[k] = v;
        const int li = own_row<T, RPT>(k);
        if (li < R)
            pv[li] = v;
    };
    auto gave_up = [&]() { a.ctl->fault = a.epoch; };
    // A p and its inner products with p and itself into acc[0], acc[1]
    auto product = [&](dd &pap, dd &apap) {
#pragma unroll
        for (int k = 0; k < RPT; ++k) {
            const double q = M.dot(k, pv);
            ap[k] = q;
            publish(k, q);
            dd_fma(pap, q, p_of(k));
            dd_fma(apap, q, q);
            if constexpr (P_LDS)
                __builtin_amdgcn_sched_barrier(0);  // one row's gathers at a time (registers)
        }
    };

    if (!a.resume) {
#pragma unroll
        for (int k = 0; k < RPT; ++k)
            if (k * T + tid < R)
                pv[k * T + tid] = row0 + k * T + tid < n ? a.x[row0 + k * T + tid] : 0.0;
        for (int j = tid; j < ng; j += T)
            pv[R + j] = a.x[gl[j]];
        __syncthreads();
        dd acc[2] = {dd{0.0, 0.0}, dd{0.0, 0.0}};
#pragma unroll
        for (int k = 0; k < RPT; ++k) {
            const int li = k * T + tid, row = row0 + li;
            const double bi = li < R && row < n ? a.b[row] : 0.0;
            const double ri = bi - M.dot(k, pv);
            rr[k] = ri;
            if constexpr (P_LDS)
                __builtin_amdgcn_sched_barrier(0);
            publish(k, ri);
            dd_fma(acc[0], ri, ri);
            dd_fma(acc[1], bi, bi);
        }
        const bool ok = all_reduce<T, 2>(acc, sh, a, g, tag, ll(), gl, ng, gw, [&](const double *d) {
            if (tid == 0)
                finalize(&sh.s, FIN_SETUP, d, 2, hist, scal);
        });
        if (!ok)
            return gave_up();
        if (sh.s.status == ST_RUNNING) {
#pragma unroll
            for (int k = 0; k < RPT; ++k)
                p_set(k, rr[k]);
            if (!each_ghost([&](int j, double v) { rg[j] = pv[R + j] = v; }))
                sh.fault = 1;
            __syncthreads();
            ++tag;
            dd acc1[2] = {dd{0.0, 0.0}, dd{0.0, 0.0}};
            product(acc1[0], acc1[1]);
            if (!all_reduce<T, 2>(acc1, sh, a, g, tag, ll(), gl, ng, gw, [&](const double *d) {
                    if (tid == 0)
                        finalize(&sh.s, FIN_CG_ALPHA, d, 2, hist, scal);
                }))
                return gave_up();
        }
    } else {
        // r, p of the ghosts from where their owners left them; A p again by words
#pragma unroll
        for (int k = 0; k < RPT; ++k) {
            const int li = k * T + tid;
            publish(k, ap[k]);
            p_set(k, li < R && row0 + li < n ? a.p[par][row0 + li] : 0.0);
        }
        for (int j = tid; j < ng; j += T) {
            rg[j] = a.r[par][gl[j]];
            pv[R + j] = a.p[par][gl[j]];
        }
        if (!ghost_poll<T>(ll(), gl, ng, tag, gw))
            sh.fault = 1;
        __syncthreads();
        if (sh.fault)
            return gave_up();
    }
    // The scalars of the loop: wave 0 of every workgroup computes them from
    // registers (FIN_CG_RR_ALPHA, the same expressions) and leaves what the
    // other waves need in LDS; the norm's square root and quotient only feed
    // the history and, near the tolerance, the test, so they stay off the path
    // between two products.
    const double bnorm = sh.s.bnorm, tol = sh.s.tol;
    const double near = tol > 1e-150 ? tol * tol * (1.0 + 1e-12) : HUGE_VAL;  // above it sqrt(rr) > tol for certain
    const int max_iter = sh.s.max_iter, it0 = sh.s.it;
    int it = it0, status = sh.s.status;
    double alpha = sh.s.alpha, beta = sh.s.beta, rr_last = sh.s.rr;
    while (status == ST_RUNNING && it - it0 < a.chunk) {
        dd acc[3] = {dd{0.0, 0.0}, dd{0.0, 0.0}, dd{0.0, 0.0}};
        // x_i, r_i, p_i and <r_i, r_i>; r_i, p_i of the ghosts
        if (!each_ghost([&](int j, double v) {
                const double ri = rg[j] - alpha * v;
                rg[j] = ri;
                pv[R + j] = ri + beta * pv[R + j];
            }))
            sh.fault = 1;
#pragma unroll
        for (int k = 0; k < RPT; ++k) {
            const double pi = p_of(k);
            if constexpr (!X_MEM) {
                xr[k] = xr[k] + alpha * pi;
            } else {
                const int li = own_row<T, RPT>(k);
                if (li < R && row0 + li < n) {
                    double *xp = reinterpret_cast<double *>(reinterpret_cast<char *>(a.x + row0) + (uint32_t)li * 8u);
                    *xp = *xp + alpha * pi;
                }
            }
            const double ri = rr[k] - alpha * ap[k];
            rr[k] = ri;
            p_set(k, ri + beta * pi);
            dd_fma(acc[2], ri, ri);
        }
        __syncthreads();
        ++tag;
        product(acc[0], acc[1]);
        if (!all_reduce<T, 3>(acc, sh, a, g, tag, ll(), gl, ng, gw, [&](const double *d) {
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
                if (tid == 0) {
                    sh.alpha = al;
                    sh.beta = be;
                    sh.status = st;
                    sh.s.rr = rr1;
                }
            }))
            return gave_up();
        ++it;
        alpha = sh.alpha;
        beta = sh.beta;
        status = sh.status;
        rr_last = sh.s.rr;
        if (tid == 0 && hist) {
            put_hist(&sh.s, hist, it, sqrt(rr_last) / bnorm);
            put_scal(&sh.s, scal, it - 1, 3, rr_last);
            if (status == ST_RUNNING) {
                put_scal(&sh.s, scal, it, 0, alpha);
                put_scal(&sh.s, scal, it, 1, beta);
            }
        }
    }
    const bool more = status == ST_RUNNING;  // the chunk ended first
    const int end = it & 1;
#pragma unroll
    for (int k = 0; k < RPT; ++k) {
        const int li = k * T + tid, row = row0 + li;
        if (li < R && row < n) {
            if constexpr (!X_MEM)
                a.x[row] = xr[k];
            if (more) {
                a.r[end][row] = rr[k];
                a.p[end][row] = p_of(k);
                a.ap[end][row] = ap[k];
            }
        }
    }
    if (g == 0 && tid == 0) {
        if (it > it0) {
            sh.s.it = it;
            sh.s.status = status;
            sh.s.alpha = alpha;
            sh.s.beta = beta;
            sh.s.last_rel = sqrt(rr_last) / bnorm;
        }
        *a.st = sh.s;
    }
}

}  // namespace

// ------------------------------------------------------------------ host

namespace {

// Static LDS of the kernels (ResShared) and a margin.
constexpr size_t RES_STATIC_LDS = 4096;

using ResKernel = void (*)(ResArgs);

// Threads and rows per thread: the fewest waves whose threads keep at most
// eight rows, since every wave joins each reduction.
struct ResBody {
    int threads, rpt;
    ResKernel cg5, cg7;
};
const ResBody BODIES[] = {
    {256, 1, k_res_cg<256, 1, 5>, k_res_cg<256, 1, 7>}, {256, 2, k_res_cg<256, 2, 5>, k_res_cg<256, 2, 7>},
    {512, 2, k_res_cg<512, 2, 5>, k_res_cg<512, 2, 7>}, {512, 4, k_res_cg<512, 4, 5>, k_res_cg<512, 4, 7>},
    {512, 8, k_res_cg<512, 8, 5>, nullptr},
};

}  // namespace

bool resident_shape(const DevCsr &A, int cus, size_t max_lds, ResShape *out)
{
    if (A.nslices <= 0 || A.max_width < 1 || A.max_width > 7 || cus < 1)
        return false;
    const int gmax = cus < RES_MAX_WG ? cus : RES_MAX_WG;
    int64_t rows = ((int64_t)A.nslices + gmax - 1) / gmax * SLICE;
    if (rows < 256)
        rows = 256;
    for (int i = 0; i < (int)(sizeof(BODIES) / sizeof(BODIES[0])); ++i) {
        const ResBody &b = BODIES[i];
        if ((int64_t)b.threads * b.rpt < rows)
            continue;
        if (A.max_width > 5 && !b.cg7)
            return false;
        const size_t lds = (size_t)rows * 8 * (1 + res_lds_values(b.rpt)) + RES_STATIC_LDS;
        if (lds + 2048 > max_lds)
            return false;
        out->body = i;
        out->rows = (int)rows;
        out->groups = (int)(((int64_t)A.n + rows - 1) / rows);
        out->gcap = (int)((max_lds - lds) / 16);
        if (out->gcap > 65534 - (int)rows)
            out->gcap = 65534 - (int)rows;
        return out->groups <= RES_MAX_WG;
    }
    return false;
}

hipError_t launch_res_plan(const DevCsr &A, const ResShape &sh, uint16_t *idx, int32_t *gcount, int32_t *glist,
                           uint8_t *pub, hipStream_t s)
{
    hipLaunchKernelGGL(k_res_plan, dim3(sh.groups), dim3(PLAN_T), 0, s, A, sh.rows, sh.gcap, idx, gcount, glist, pub);
    return hipGetLastError();
}

hipError_t launch_res_cg(const ResShape &sh, const ResArgs &a, hipStream_t s)
{
    const ResBody &b = BODIES[sh.body];
    const size_t lds = ((size_t)sh.rows * (1 + res_lds_values(b.rpt)) + 2 * (size_t)sh.ghosts) * 8;
    hipLaunchKernelGGL(a.A.max_width <= 5 ? b.cg5 : b.cg7, dim3(sh.groups), dim3(b.threads), (uint32_t)lds, s, a);
    return hipGetLastError();
}

}  // namespace fk
