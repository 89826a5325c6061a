// The bottom of a V-cycle in one workgroup.  Below a few thousand rows a
// launch moves less data than it takes to start: each of a level's six
// launches runs 2.5 to 4 us for well under 1 us of work.  Here one workgroup
// takes one right-hand side (or one system of a batch) from the first small
// level down to the coarsest solve and back, its vectors in LDS, with a
// barrier where the launches had a kernel boundary.
//
// What bounds it is the chain from barrier to barrier (about 0.7 us a phase at
// a few hundred rows: gather, lane sums, division, LDS store) and, at a few
// thousand rows, the instructions of one CU.  So the operators are packed for
// the lanes that sum them (TailSet): a chunk's addresses follow from its
// number, its loads need no row pointer and are issued a phase ahead, across
// the barrier, and unused places multiply a zero instead of being asked for.
// A cycle on a 64 x 64 grid in FP64: 85 to 95 us in 29 launches, 47 us here
// with CSR rows, 38 us packed (1,024 threads; 62 us with 512).
//
// Every row is summed by as many lanes, over the same entries in the same
// order, as in the launches of k_cycle.hip, so the results are theirs bit for
// bit.
#include <algorithm>
#include <cmath>
#include <cstddef>
#include <type_traits>
#include <vector>

#include "k_common.hpp"
#include "lair_internal.hpp"
#include "tail.hpp"

namespace lair {

constexpr int TAIL_BS = 1024;
constexpr int TAIL_WAVES = TAIL_BS / WAVE;

size_t tail_layout(TailSet &t, size_t at, int32_t nchunk, bool rows, size_t w) {
    const size_t entries = (size_t)nchunk * t.smax * WAVE * (t.u4 ? 4 : 1);
    size_t o = at;
    t.o_used = (uint32_t)o;
    o += ((size_t)nchunk * 2 + 15) & ~(size_t)15;
    t.o_row = (uint32_t)o;
    if (rows) o += (size_t)nchunk * WAVE * 2;
    t.o_diag = (uint32_t)o;
    if (rows) o += (size_t)nchunk * WAVE * w;
    t.o_col = (uint32_t)o;
    o += entries * 2;
    t.o_val = (uint32_t)o;
    o += entries * w;
    return (o + 255) & ~(size_t)255;
}

int32_t tail_groups(int32_t max_row, int lg, int ll, bool u4) {
    const int step = 1 << (lg + ll);
    const int share = (max_row + step - 1) / step << ll;
    const int U = u4 ? 4 : 1;
    return std::max(1, (share + U - 1) / U);
}

// Entry m of lane g's share: steps of 2^(lg + ll) entries, of which the lane
// takes 2^ll consecutive ones.
__device__ __forceinline__ int share_pos(int lo, int g, int m, int lg, int ll) {
    return lo + ((m >> ll) << (lg + ll)) + (g << ll) + (m & ((1 << ll) - 1));
}

// ---------------------------------------------------------------------------
// Packing: one wave per chunk, the sets of all levels in one launch.  It is
// part of a hierarchy's first cycle and of the first after a new diagonal, and
// bound by latency: its launches (one a level before) and, in rows of some
// hundred entries, one load after another (before: the diagonal looked for in
// every entry, the entries copied one by one).  So the diagonal is found by
// halves, and a lane fetches PACK_K entries at a time.  First cycle of a
// 66 x 66 grid 133 -> 109 us, of a 1000-row arrow matrix
// 495 -> 255, of 3000 rows with three of 500 entries 350 -> 190.
// ---------------------------------------------------------------------------
constexpr int PACK_BS = 256;
constexpr int PACK_SETS = 32;       // the table is a kernel argument (4 KB)
constexpr int PACK_K = 16;

template <class VT>
struct PackArgs {
    char *blob;
    int32_t nset;
    int32_t block0[PACK_SETS + 1];  // each set's first block
    TailSource<VT> src[PACK_SETS];
};

template <class VT>
__global__ void __launch_bounds__(PACK_BS)
k_tail_pack(const PackArgs<VT> t) {
    static_assert(sizeof(PackArgs<VT>) <= 4096, "");
    int set = 0;
    for (int q = 1; q < t.nset; ++q) set += (int)blockIdx.x >= t.block0[q] ? 1 : 0;
    const TailSource<VT> &S = t.src[set];
    const int ch = ((int)blockIdx.x - t.block0[set]) * (PACK_BS / WAVE) + threadIdx.x / WAVE;
    if (ch >= S.nchunk) return;
    const int lane = threadIdx.x & (WAVE - 1);
    const int lg = S.lg, ll = S.ll, g = lane & ((1 << lg) - 1);
    const bool u4 = S.dst.u4;
    const int U = u4 ? 4 : 1, smax = S.dst.smax;
    // the chunk's system, its first row (or list position) and its columns' base
    int k = (ch << (6 - lg)) + (lane >> lg), hi_k = S.n, ncol = S.ncol;
    int64_t base = 0, c0 = 0, rb = 0;
    if (S.chunk0) {
        int lo = 0, hi = S.nsys - 1;
        while (lo < hi) {
            const int mid = (lo + hi + 1) >> 1;
            if (S.chunk0[mid] <= ch) lo = mid; else hi = mid - 1;
        }
        rb = S.rseg[lo];
        base = S.rows ? S.run[lo] : rb;
        c0 = S.cseg[lo];
        ncol = (int)(S.cseg[lo + 1] - c0);
        k -= S.chunk0[lo] << (6 - lg);
        hi_k = S.rows ? S.run[lo + 1] - S.run[lo] : (int)(S.rseg[lo + 1] - rb);
    }
    const int32_t *cj = S.cj;
    const VT *v = S.v;
    int i = 0, p0 = 0, p1 = 0;
    if (k < hi_k) {
        i = S.rows ? S.rows[base + k] : (int)(base + k);
        p0 = S.rp[i];
        p1 = S.rp[i + 1];
    }
    // entries of this lane's share: whole steps, and its part of the last one
    const int step = lg + ll, rest = (p1 - p0) & ((1 << step) - 1);
    const int mine = (((p1 - p0) >> step) << ll) + min(max(rest - (g << ll), 0), 1 << ll);
    int ng = (mine + U - 1) / U;
#pragma unroll
    for (int o = WAVE / 2; o > 0; o >>= 1) ng = max(ng, __shfl_xor(ng, o));
    ng = min(ng, smax);
    char *blob = t.blob;
    if (lane == 0) reinterpret_cast<uint16_t *>(blob + S.dst.o_used)[ch] = (uint16_t)ng;
    if (S.diag) {
        const int p = bsearch_i32(cj + p0, p1 - p0, i);
        reinterpret_cast<uint16_t *>(blob + S.dst.o_row)[(size_t)ch * WAVE + lane] =
            k < hi_k ? (uint16_t)(i - rb) : (uint16_t)0;
        reinterpret_cast<VT *>(blob + S.dst.o_diag)[(size_t)ch * WAVE + lane] =
            p >= 0 ? v[p0 + p] : (VT)0;
    }
    uint16_t *col = reinterpret_cast<uint16_t *>(blob + S.dst.o_col);
    VT *val = reinterpret_cast<VT *>(blob + S.dst.o_val);
    const int entries = max(ng, 1) * U;
    for (int m0 = 0; m0 < entries; m0 += PACK_K) {
        int c[PACK_K];
        VT a[PACK_K];
#pragma unroll
        for (int u = 0; u < PACK_K; ++u) {
            const int p = share_pos(p0, g, m0 + u, lg, ll);
            c[u] = p < p1 ? (int)(cj[p] - c0) : ncol;
            a[u] = p < p1 ? v[p] : (VT)0;
        }
#pragma unroll
        for (int u = 0; u < PACK_K; ++u) {
            const int m = m0 + u;
            if (m >= entries) break;
            const size_t o = (((size_t)ch * smax + m / U) * WAVE + lane) * U + m % U;
            col[o] = (uint16_t)c[u];
            val[o] = a[u];
        }
    }
}

template <class VT>
void launch_tail_pack(const std::vector<TailSources<VT>> &levels, hipStream_t s) {
    PackArgs<VT> t{};
    auto flush = [&] {
        if (t.nset == 0) return;
        LAIR_LAUNCH((k_tail_pack<VT>), dim3((unsigned)t.block0[t.nset]), dim3(PACK_BS), 0, s, t);
        LAIR_LAUNCH_CHECK();
        t.nset = 0;
    };
    for (const auto &level : levels)
        for (const auto &S : level.src) {
            if (S.nchunk == 0) continue;
            t.blob = level.blob;
            t.src[t.nset] = S;
            t.block0[t.nset + 1] =
                t.block0[t.nset] + (int32_t)blocks_for(S.nchunk, PACK_BS / WAVE);
            if (++t.nset == PACK_SETS) flush();
        }
    flush();
}

// ---------------------------------------------------------------------------
// The tail
// ---------------------------------------------------------------------------
// Barrier ordering LDS only: global loads stay in flight across it (what
// they read is not written by this kernel).
__device__ __forceinline__ void lds_barrier() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// A row set of one level for one system: the parts of its blob (byte
// addresses, the system's first chunk applied) and its rows.
// (addresses read from a table: the compiler must be told that they are in
// global memory, or it loads through the flat path, which counts against LDS
// and stalls the barriers)
#define LAIR_GLOBAL __attribute__((address_space(1)))
using GlobalBytes = const LAIR_GLOBAL char *;
struct RowSet {
    GlobalBytes used, row, diag, col, val;
    int n, lg, smax;
    bool u4;
};

using u32x2 = ExtVec<uint32_t, 2>;

// Four entries of a lane's share (columns packed two to a word).
template <class VT>
struct Group {
    uint32_t c01, c23;
    VT a0, a1, a2, a3;
};

// The first group of a lane's share in one chunk.
template <class VT>
struct Head {
    Group<VT> g;
    VT d;
    int row, used;
};

template <class VT, bool U4>
__device__ __forceinline__ Group<VT> load_group(const RowSet &S, int ch, int grp) {
    Group<VT> G{};
    const uint32_t lane = threadIdx.x & (WAVE - 1);
    const uint32_t o = (uint32_t)(ch * S.smax + grp) * WAVE + lane;
    if (U4) {
        const u32x2 cc = *reinterpret_cast<const LAIR_GLOBAL u32x2 *>(S.col + (size_t)(o * 8u));
        G.c01 = cc.x;
        G.c23 = cc.y;
        GlobalBytes pv = S.val + (size_t)(o * (uint32_t)(4 * sizeof(VT)));
        if constexpr (sizeof(VT) == 4) {
            const ExtVec<float, 4> v = *reinterpret_cast<const LAIR_GLOBAL ExtVec<float, 4> *>(pv);
            G.a0 = v.x;
            G.a1 = v.y;
            G.a2 = v.z;
            G.a3 = v.w;
        } else {
            const ExtVec<double, 2> v0 = reinterpret_cast<const LAIR_GLOBAL ExtVec<double, 2> *>(pv)[0];
            const ExtVec<double, 2> v1 = reinterpret_cast<const LAIR_GLOBAL ExtVec<double, 2> *>(pv)[1];
            G.a0 = v0.x;
            G.a1 = v0.y;
            G.a2 = v1.x;
            G.a3 = v1.y;
        }
    } else {
        G.c01 = *reinterpret_cast<const LAIR_GLOBAL uint16_t *>(S.col + (size_t)(o * 2u));
        G.a0 = *reinterpret_cast<const LAIR_GLOBAL VT *>(S.val + (size_t)(o * (uint32_t)sizeof(VT)));
    }
    return G;
}

// Unused entries have value 0 and the column of the zero that follows the
// source vector, so nothing is asked per entry.
template <class VT, bool U4>
__device__ __forceinline__ void add_group(const Group<VT> &G, const VT *src, VT &acc) {
    if (U4) {
        const VT x0 = src[G.c01 & 0xffffu], x1 = src[G.c01 >> 16];
        const VT x2 = src[G.c23 & 0xffffu], x3 = src[G.c23 >> 16];
        acc += G.a0 * x0;
        acc += G.a1 * x1;
        acc += G.a2 * x2;
        acc += G.a3 * x3;
    } else {
        acc += G.a0 * src[G.c01];
    }
}

// Chunk ch of the set, if it has one (a wave-uniform question).
template <class VT, bool DIAG, bool U4>
__device__ __forceinline__ void load_head(const RowSet &S, int ch, Head<VT> &h) {
    if (ch << (6 - S.lg) >= S.n) return;
    const uint32_t o = (uint32_t)ch * WAVE + (threadIdx.x & (WAVE - 1));
    h.used = *reinterpret_cast<const LAIR_GLOBAL uint16_t *>(S.used + 2 * (size_t)ch);
    if (DIAG) {
        h.row = *reinterpret_cast<const LAIR_GLOBAL uint16_t *>(S.row + (size_t)(o * 2u));
        h.d = *reinterpret_cast<const LAIR_GLOBAL VT *>(S.diag + (size_t)(o * (uint32_t)sizeof(VT)));
    }
    h.g = load_group<VT, U4>(S, ch, 0);
}

__device__ __forceinline__ int wave_id() {
    return __builtin_amdgcn_readfirstlane(threadIdx.x / WAVE);
}

// One chunk: each row's product with src (LDS), then fin(k, row, acc, d) on
// its team's first lane, k the row's place in the set.
template <class VT, bool MULTI, bool GATHER, bool U4, class Fin>
__device__ __forceinline__ void one_chunk(const RowSet &S, int ch, const Head<VT> &h,
                                          const VT *src, Fin &&fin) {
    const int lane = threadIdx.x & (WAVE - 1);
    const int G = 1 << S.lg;
    VT acc = (VT)0;
    if (GATHER) {
        add_group<VT, U4>(h.g, src, acc);
        const int used = __builtin_amdgcn_readfirstlane(h.used);
        for (int grp = 1; grp < used; ++grp)
            add_group<VT, U4>(load_group<VT, U4>(S, ch, grp), src, acc);
        if (MULTI)
            for (int o = 1; o < G; o <<= 1) acc += __shfl_xor(acc, o);
        else
            for (int o = G >> 1; o > 0; o >>= 1) acc += __shfl_xor(acc, o);
    }
    const int k = (ch << (6 - S.lg)) + (lane >> S.lg);
    if ((lane & (G - 1)) == 0 && k < S.n) fin(k, h.row, acc, h.d);
}

// The rows of set S, a wave's chunks in turn; h: its first chunk, loaded in
// the phase before; each further chunk is loaded one ahead.  MULTI: the sums
// of several right-hand sides (lane partial sums added from the nearest lane
// out), else those of one (from the farthest in).  Without GATHER the product
// is zero (a zero source).
template <class VT, bool MULTI, bool DIAG, bool GATHER, bool U4, class Fin>
__device__ __forceinline__ void set_phase(const RowSet &S, Head<VT> h, const VT *src,
                                          Fin &&fin) {
    const int nch = (S.n + (WAVE >> S.lg) - 1) >> (6 - S.lg);
    Head<VT> h1;
    for (int ch = wave_id(); ch < nch; ch += 2 * TAIL_WAVES) {
        load_head<VT, DIAG, U4>(S, ch + TAIL_WAVES, h1);
        one_chunk<VT, MULTI, GATHER, U4>(S, ch, h, src, fin);
        if (ch + TAIL_WAVES >= nch) break;
        load_head<VT, DIAG, U4>(S, ch + 2 * TAIL_WAVES, h);
        one_chunk<VT, MULTI, GATHER, U4>(S, ch + TAIL_WAVES, h1, src, fin);
    }
}

// Sets whose rows have one entry per lane (one-point interpolation) are
// stored without groups of four.
template <class VT>
__device__ __forceinline__ void load_ahead_p(const RowSet &S, Head<VT> &h) {
    if (S.u4) load_head<VT, false, true>(S, wave_id(), h);
    else load_head<VT, false, false>(S, wave_id(), h);
}
template <class VT, bool DIAG>
__device__ __forceinline__ void load_ahead(const RowSet &S, Head<VT> &h) {
    load_head<VT, DIAG, true>(S, wave_id(), h);
}

template <class VT, bool MULTI, class Fin>
__device__ __forceinline__ void row_phase_p(const RowSet &S, const Head<VT> &h, const VT *src,
                                            Fin &&fin) {
    if (S.u4) set_phase<VT, MULTI, false, true, true>(S, h, src, fin);
    else set_phase<VT, MULTI, false, true, false>(S, h, src, fin);
}
template <class VT, bool MULTI, bool DIAG, bool GATHER = true, class Fin>
__device__ __forceinline__ void row_phase(const RowSet &S, const Head<VT> &h, const VT *src,
                                          Fin &&fin) {
    set_phase<VT, MULTI, DIAG, GATHER, true>(S, h, src, fin);
}

__device__ __forceinline__ int uniform(int v) { return __builtin_amdgcn_readfirstlane(v); }
template <class T>
__device__ __forceinline__ T *uniform_ptr(T *p) {
    const uint64_t u = reinterpret_cast<uint64_t>(p);
    const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)u);
    const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)(u >> 32));
    return reinterpret_cast<T *>((uint64_t)hi << 32 | lo);
}

// x = M b for the dense m x m inverse M (rows, or columns with TRANS), TC
// lanes per output, in double whatever the vector type.
template <class VT, int TC, bool TRANS>
__device__ __forceinline__ void dense_phase(int m, const double *Mp, const VT *b, VT *x) {
    const LAIR_GLOBAL double *M = (const LAIR_GLOBAL double *)uniform_ptr(Mp);
    m = uniform(m);
    const int lane = threadIdx.x % TC;
    for (int i = threadIdx.x / TC; i < m; i += TAIL_BS / TC) {
        double acc = 0.0;
#pragma unroll 8
        for (int j = lane; j < m; j += TC)
            acc += (TRANS ? M[(size_t)j * m + i] : M[(size_t)i * m + j]) * (double)b[j];
        acc = team_sum<TC>(acc);
        if (lane == 0) x[i] = (VT)acc;
    }
}

// The argument table in LDS, read by every lane at once: a table lives in
// kernel argument memory, where each line's first scalar load takes about a
// microsecond, and a cycle would meet some forty of them one after another.
template <class VT>
__device__ __forceinline__ void stage_args(const TailArgs<VT> &a, TailArgs<VT> &s) {
    static_assert(sizeof(TailArgs<VT>) % 8 == 0 && sizeof(TailArgs<VT>) <= 8 * TAIL_BS, "");
    const size_t words = (offsetof(TailArgs<VT>, lv) + (size_t)a.nlv * sizeof(TailLevel<VT>)) / 8;
    if (threadIdx.x < words)
        reinterpret_cast<uint64_t *>(&s)[threadIdx.x] =
            reinterpret_cast<const uint64_t *>(&a)[threadIdx.x];
    __syncthreads();
}

// The system's (or the single system's) place on every level.
struct TailMap {
    int n[TAIL_MAX_LEVELS], row0[TAIL_MAX_LEVELS], off[TAIL_MAX_LEVELS];
    int nset[TAIL_SETS][TAIL_MAX_LEVELS], ch0[TAIL_SETS][TAIL_MAX_LEVELS];
};

// off: where each level's vector lies in LDS (a zero after each), after two
// vectors of the first level and, with before = 3, one of the second.
template <class VT>
__device__ __forceinline__ void tail_map(const TailArgs<VT> &a, int q, int top, int last,
                                         int before, TailMap &m) {
    if ((int)threadIdx.x < a.nlv) {
        const int l = threadIdx.x;
        const TailLevel<VT> &L = a.lv[l];
        const bool batch = L.seg != nullptr;
        m.row0[l] = batch ? (int)L.seg[q] : 0;
        const int n = batch ? (int)(L.seg[q + 1] - L.seg[q]) : L.n;
        m.n[l] = n;
        m.nset[TAIL_P][l] = m.nset[TAIL_A][l] = n;
        if (l + 1 < a.nlv) {
            m.nset[TAIL_F][l] = batch ? L.frun[q + 1] - L.frun[q] : L.nf;
            m.nset[TAIL_C][l] = batch ? L.crun[q + 1] - L.crun[q] : L.nc;
            const int64_t *sn = a.lv[l + 1].seg;
            m.nset[TAIL_R][l] = batch ? (int)(sn[q + 1] - sn[q]) : a.lv[l + 1].n;
            for (int t = 0; t < TAIL_SETS; ++t)
                m.ch0[t][l] = batch ? L.chunk0[t * (a.nsys + 1) + q] : 0;
        }
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        int o = 2 * (m.n[top] + 1) + (before == 3 && top < last ? m.n[top + 1] + 1 : 0);
        for (int l = top; l <= last; ++l) {
            m.off[l] = o;
            o += m.n[l] + 1;
        }
    }
    __syncthreads();
}

template <class VT>
__device__ __forceinline__ RowSet row_set(const TailArgs<VT> &a, const TailMap &m, int l, int t) {
    const TailSet &T = a.lv[l].set[t];
    GlobalBytes blob = (GlobalBytes)uniform_ptr(a.blob);
    RowSet S;
    S.lg = uniform(T.lg);
    S.smax = uniform(T.smax);
    S.u4 = uniform(T.u4) != 0;
    S.n = uniform(m.nset[t][l]);
    const uint32_t ch0 = uniform(m.ch0[t][l]), lanes = ch0 * WAVE;
    const uint32_t slots = lanes * S.smax * (S.u4 ? 4 : 1);
    S.used = blob + (uint32_t)uniform(T.o_used) + (size_t)(ch0 * 2u);
    S.row = blob + (uint32_t)uniform(T.o_row) + (size_t)lanes * 2;
    S.diag = blob + (uint32_t)uniform(T.o_diag) + (size_t)lanes * sizeof(VT);
    S.col = blob + (uint32_t)uniform(T.o_col) + (size_t)slots * 2;
    S.val = blob + (uint32_t)uniform(T.o_val) + (size_t)slots * sizeof(VT);
    return S;
}

// LDS: the iterate and a sweep buffer of the first level's size (every level
// uses them in turn), then the right-hand side of each level and the coarsest
// solution.  On the way up a level's result takes its right-hand side's
// place: the sweeps read b only at the row they write.
template <class VT, bool MULTI, int MODE, bool BATCH>
__global__ void __launch_bounds__(TAIL_BS)
k_tail(const TailArgs<VT> args, const VT *b, VT *x, const VT *r) {
    extern __shared__ __align__(16) char tail_lds[];
    __shared__ TailMap mp;
    __shared__ TailArgs<VT> a;
    if (BATCH && args.active && !args.active[args.order[blockIdx.x]]) return;
    stage_args(args, a);
    VT *const W = reinterpret_cast<VT *>(tail_lds);
    const int q = BATCH ? uniform(args.order[blockIdx.x]) : 0;
    const int rhs = BATCH ? 0 : blockIdx.x, R = BATCH ? 1 : args.nrhs;
    const int top = BATCH ? uniform(args.top[q]) : 0;
    const int last = (BATCH ? uniform(args.slev[q]) : args.nlv) - 1;
    tail_map(a, q, top, last, 2, mp);
    const int n0 = uniform(mp.n[top]), r0 = uniform(mp.row0[top]);
    VT *const X = W, *const Y = W + n0 + 1, *const B0 = W + 2 * (n0 + 1);
    // the zeros after the vectors (a level's X and Y end at its own size: see
    // the interpolation)
    for (int l = top + threadIdx.x; l <= last; l += TAIL_BS) {
        W[mp.off[l] + mp.n[l]] = (VT)0;
        if (l == last) W[mp.off[l] + 2 * mp.n[l] + 1] = (VT)0;
    }
    if (threadIdx.x == 0) X[n0] = Y[n0] = (VT)0;
    const LAIR_GLOBAL VT *bt = (const LAIR_GLOBAL VT *)uniform_ptr(BATCH ? a.lv[top].vb : b);
    LAIR_GLOBAL VT *xt = (LAIR_GLOBAL VT *)uniform_ptr(BATCH ? a.lv[top].vx : x);
    Head<VT> p;
    RowSet S;
    if (top < last) {
        S = row_set(a, mp, top, MODE == TAIL_ITERATE ? TAIL_A : TAIL_R);
        load_ahead<VT, false>(S, p);
    }
    for (int i = threadIdx.x; i < n0; i += TAIL_BS) {
        const size_t gi = (size_t)(r0 + i) * R + rhs;
        B0[i] = bt[gi];
        if (MODE == TAIL_ITERATE) X[i] = xt[gi];
        if (MODE == TAIL_RESID) Y[i] = r[gi];
    }
    if (MODE == TAIL_ITERATE) {
        const RowSet SR = row_set(a, mp, top, TAIL_R);
        Head<VT> pr;
        lds_barrier();
        load_ahead<VT, false>(SR, pr);
        row_phase<VT, MULTI, false>(S, p, X, [&](int k, int, VT acc, VT) { Y[k] = B0[k] - acc; });
        S = SR;
        p = pr;
    }
    for (int l = top; l < last; ++l) {
        // the next set: the restriction below, or the first interpolation
        const bool down = l + 1 < last;
        const RowSet SN = row_set(a, mp, down ? l + 1 : l, down ? TAIL_R : TAIL_P);
        const VT *src = (MODE != TAIL_ZERO && l == top) ? Y : W + uniform(mp.off[l]);
        VT *dst = W + uniform(mp.off[l + 1]);
        Head<VT> pn;
        lds_barrier();
        if (down) load_ahead<VT, false>(SN, pn);
        else load_ahead_p<VT>(SN, pn);
        row_phase<VT, MULTI, false>(S, p, src, [&](int k, int, VT acc, VT) { dst[k] = acc; });
        S = SN;
        p = pn;
    }
    {
        const int m = uniform(mp.n[last]);
        VT *bl = W + uniform(mp.off[last]), *out = bl + m + 1;
        lds_barrier();
        if (BATCH) dense_phase<VT, WAVE, false>(m, a.binv + a.doff[q], bl, out);
        else dense_phase<VT, 16, false>(m, a.kinv, bl, out);
    }
    const VT om = a.omega;
    for (int l = last - 1; l >= top; --l) {
        VT *bl = W + uniform(mp.off[l]);
        const VT *e = W + uniform(mp.off[l + 1] + (l + 1 == last ? mp.n[last] + 1 : 0));
        const bool add = MODE != TAIL_ZERO && l == top;
        const RowSet SF = row_set(a, mp, l, TAIL_F);
        if (args.knode) {
            // the sweeps' right-hand side D^{-1} b
            const int kn = args.knode, n = uniform(mp.n[l]);
            const LAIR_GLOBAL double *dinv =
                (const LAIR_GLOBAL double *)uniform_ptr(a.lv[l].dinv);
            lds_barrier();
            for (int i = threadIdx.x; i < n; i += TAIL_BS) {
                const LAIR_GLOBAL double *d = dinv + (size_t)i * kn;
                const VT *bb = bl + i / kn * kn;
                double acc = 0.0;
                for (int c = 0; c < kn; ++c) acc += d[c] * (double)bb[c];
                Y[i] = (VT)acc;
            }
            lds_barrier();
            for (int i = threadIdx.x; i < n; i += TAIL_BS) bl[i] = Y[i];
        }
        Head<VT> pf;
        lds_barrier();
        load_ahead<VT, true>(SF, pf);
        if (threadIdx.x == 0) X[mp.n[l]] = Y[mp.n[l]] = (VT)0;
        row_phase_p<VT, MULTI>(S, p, e, [&](int k, int, VT acc, VT) {
            const VT xv = add ? xt[(size_t)(r0 + k) * R + rhs] + acc : acc;
            X[k] = xv;
            Y[k] = xv;
        });
        // F sweep: reads X, writes Y at the F rows (Y holds X at the C rows)
        const RowSet SC = row_set(a, mp, l, TAIL_C);
        lds_barrier();
        row_phase<VT, MULTI, true>(SF, pf, X, [&](int, int i, VT acc, VT d) {
            Y[i] = X[i] + om * (bl[i] - acc) / d;
        });
        Head<VT> pc;
        lds_barrier();
        load_ahead<VT, true>(SC, pc);
        row_phase<VT, MULTI, true>(SF, pf, Y, [&](int, int i, VT acc, VT d) {
            const VT xv = Y[i] + om * (bl[i] - acc) / d;
            X[i] = xv;
            bl[i] = xv;
        });
        lds_barrier();
        if (l > top) {
            S = row_set(a, mp, l - 1, TAIL_P);
            load_ahead_p<VT>(S, p);
        }
        row_phase<VT, MULTI, true>(SC, pc, X, [&](int, int i, VT acc, VT d) {
            bl[i] = X[i] + om * (bl[i] - acc) / d;
        });
    }
    lds_barrier();
    const VT *out = top == last ? B0 + n0 + 1 : B0;
    for (int i = threadIdx.x; i < n0; i += TAIL_BS) xt[(size_t)(r0 + i) * R + rhs] = out[i];
}

// The transposed tail from a zero iterate: per level C, F, F sweeps, the
// residual (in the right-hand side's place) and its restriction on the way
// down, the correction added on the way up.  LDS: a sweep buffer of the first
// level's size, two right-hand sides in turn, every level's iterate.
template <bool MULTI>
__global__ void __launch_bounds__(TAIL_BS)
k_tail_t(const TailArgs<double> args, const double *g, double *lam) {
    extern __shared__ __align__(16) char tail_lds[];
    __shared__ TailMap mp;
    __shared__ TailArgs<double> a;
    stage_args(args, a);
    double *const W = reinterpret_cast<double *>(tail_lds);
    const int rhs = blockIdx.x, R = args.nrhs, last = args.nlv - 1;
    tail_map(a, 0, 0, last, 3, mp);
    const int n0 = uniform(mp.n[0]);
    double *const Y = W, *const Ba = W + n0 + 1, *const Bb = W + 2 * (n0 + 1);
    RowSet SC = row_set(a, mp, 0, TAIL_C);
    Head<double> pc;
    load_ahead<double, true>(SC, pc);
    for (int i = threadIdx.x; i < n0; i += TAIL_BS) Ba[i] = g[(size_t)i * R + rhs];
    const double om = a.omega;
    for (int l = 0; l < last; ++l) {
        double *X = W + uniform(mp.off[l]), *bl = l & 1 ? Bb : Ba, *bn = l & 1 ? Ba : Bb;
        const RowSet SF = row_set(a, mp, l, TAIL_F);
        const int n = uniform(mp.n[l]);
        for (int i = threadIdx.x; i <= n; i += TAIL_BS) X[i] = 0.0;
        if (threadIdx.x == 0) Y[n] = bl[n] = 0.0;
        Head<double> pf, pa, pr;
        lds_barrier();
        load_ahead<double, true>(SF, pf);
        // the iterate is zero: the C sweep needs the diagonal alone
        row_phase<double, MULTI, true, false>(SC, pc, X, [&](int, int i, double acc, double d) {
            const double xv = 0.0 + om * (bl[i] - acc) / d;
            X[i] = xv;
            Y[i] = xv;
        });
        const RowSet SA = row_set(a, mp, l, TAIL_A);
        lds_barrier();
        row_phase<double, MULTI, true>(SF, pf, X, [&](int, int i, double acc, double d) {
            Y[i] = X[i] + om * (bl[i] - acc) / d;
        });
        lds_barrier();
        load_ahead<double, false>(SA, pa);
        row_phase<double, MULTI, true>(SF, pf, Y, [&](int, int i, double acc, double d) {
            X[i] = Y[i] + om * (bl[i] - acc) / d;
        });
        const RowSet SR = row_set(a, mp, l, TAIL_R);
        lds_barrier();
        load_ahead<double, false>(SR, pr);
        row_phase<double, MULTI, false>(SA, pa, X, [&](int k, int, double acc, double) {
            bl[k] = bl[k] - acc;
        });
        lds_barrier();
        if (l + 1 < last) {
            SC = row_set(a, mp, l + 1, TAIL_C);
            load_ahead<double, true>(SC, pc);
        }
        row_phase<double, MULTI, false>(SR, pr, bl, [&](int k, int, double acc, double) {
            bn[k] = acc;
        });
    }
    RowSet SP = row_set(a, mp, std::max(last - 1, 0), TAIL_P);
    Head<double> pp;
    if (last > 0) load_ahead_p<double>(SP, pp);
    lds_barrier();
    dense_phase<double, 16, true>(mp.n[last], a.kinv, last & 1 ? Bb : Ba, W + mp.off[last]);
    if (threadIdx.x == 0) W[mp.off[last] + mp.n[last]] = 0.0;
    for (int l = last - 1; l >= 0; --l) {
        double *X = W + uniform(mp.off[l]);
        const double *e = W + uniform(mp.off[l + 1]);
        const RowSet SN = row_set(a, mp, std::max(l - 1, 0), TAIL_P);
        Head<double> pn;
        lds_barrier();
        if (l > 0) load_ahead_p<double>(SN, pn);
        row_phase_p<double, MULTI>(SP, pp, e, [&](int k, int, double acc, double) {
            X[k] += acc;
        });
        SP = SN;
        pp = pn;
    }
    lds_barrier();
    const double *x0 = W + mp.off[0];
    for (int i = threadIdx.x; i < n0; i += TAIL_BS) lam[(size_t)i * R + rhs] = x0[i];
}

size_t tail_lds_limit() {
    const size_t all = max_lds_per_block(), fixed = sizeof(TailMap) + sizeof(TailArgs<double>) + 64;
    return all > fixed ? all - fixed : 0;
}

template <class VT>
void launch_tail(const TailArgs<VT> &a, int mode, const VT *b, VT *x, const VT *r,
                 hipStream_t s) {
    const bool multi = a.nrhs > 1;
#define LAIR_TAIL(MU, MO, BA, NB)                                                             \
    LAIR_LAUNCH((k_tail<VT, MU, MO, BA>), dim3(NB), dim3(TAIL_BS), (size_t)a.lds_bytes, s, a, \
                b, x, r)
    if (a.order) {
        LAIR_TAIL(false, TAIL_ZERO, true, a.nsys);
    } else if (mode == TAIL_ZERO) {
        if (multi) LAIR_TAIL(true, TAIL_ZERO, false, a.nrhs);
        else LAIR_TAIL(false, TAIL_ZERO, false, 1);
    } else if constexpr (std::is_same<VT, double>::value) {
        if (mode == TAIL_RESID) {
            if (multi) LAIR_TAIL(true, TAIL_RESID, false, a.nrhs);
            else LAIR_TAIL(false, TAIL_RESID, false, 1);
        } else {
            if (multi) LAIR_TAIL(true, TAIL_ITERATE, false, a.nrhs);
            else LAIR_TAIL(false, TAIL_ITERATE, false, 1);
        }
    } else {
        fail(LAIR_EINVAL, "a float cycle starts from zero");
    }
#undef LAIR_TAIL
    LAIR_LAUNCH_CHECK();
}

void launch_tail_t(const TailArgs<double> &a, const double *g, double *lam, hipStream_t s) {
    if (a.nrhs > 1)
        LAIR_LAUNCH((k_tail_t<true>), dim3(a.nrhs), dim3(TAIL_BS), (size_t)a.lds_bytes, s, a, g,
                    lam);
    else
        LAIR_LAUNCH((k_tail_t<false>), dim3(1), dim3(TAIL_BS), (size_t)a.lds_bytes, s, a, g, lam);
    LAIR_LAUNCH_CHECK();
}

// ---------------------------------------------------------------------------
// Longest rows (of operators whose rows the setup has not measured)
// ---------------------------------------------------------------------------
struct RowPtrs {
    const int32_t *rp[3 * TAIL_MAX_LEVELS];
    int32_t n[3 * TAIL_MAX_LEVELS];
};

__global__ void __launch_bounds__(1024) k_max_rows(const RowPtrs t, int32_t *out) {
    __shared__ int32_t sh[1024];
    const int32_t *rp = t.rp[blockIdx.x];
    const int32_t n = t.n[blockIdx.x];
    int32_t m = 0;
    for (int32_t i = threadIdx.x; i < n; i += 1024) m = max(m, rp[i + 1] - rp[i]);
    sh[threadIdx.x] = m;
    __syncthreads();
    for (int o = 512; o > 0; o >>= 1) {
        if ((int)threadIdx.x < o) sh[threadIdx.x] = max(sh[threadIdx.x], sh[threadIdx.x + o]);
        __syncthreads();
    }
    if (threadIdx.x == 0) out[blockIdx.x] = sh[0];
}

void max_rows(int m, const int32_t *const *rp, const int32_t *nrows, int32_t *out,
              hipStream_t s) {
    if (m == 0) return;
    if (m > 3 * TAIL_MAX_LEVELS) fail(LAIR_EINVAL, "max_rows: %d matrices", m);
    RowPtrs t{};
    for (int k = 0; k < m; ++k) {
        t.rp[k] = rp[k];
        t.n[k] = nrows[k];
    }
    DevArr<int32_t> d;
    d.alloc((size_t)m, s);
    LAIR_LAUNCH(k_max_rows, dim3(m), dim3(1024), 0, s, t, d.get());
    LAIR_LAUNCH_CHECK();
    Readback rb(s);
    rb.add(out, d.get(), sizeof(int32_t) * m);
    rb.run();
}

template void launch_tail_pack<double>(const std::vector<TailSources<double>> &, hipStream_t);
template void launch_tail_pack<float>(const std::vector<TailSources<float>> &, hipStream_t);
template void launch_tail<double>(const TailArgs<double> &, int, const double *, double *,
                                  const double *, hipStream_t);
template void launch_tail<float>(const TailArgs<float> &, int, const float *, float *,
                                 const float *, hipStream_t);

}  // namespace lair
