// liblair cycles and solves: the V-cycle schedule (coarse-grid correction,
// then F, F, C Jacobi), its transpose, the outer iterations (stationary,
// flexible GMRES, per-system batch) and their HIP graphs.  Every arithmetic
// step runs in the HIP kernels of k_cycle.hip, k_krylov.hip and k_batch.hip.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <array>
#include <climits>
#include <cmath>
#include <cstring>
#include <memory>
#include <string>
#include <vector>

#include "hierarchy.hpp"
#include "tail.hpp"

namespace lair {

__global__ void k_add(double *x, const double *e, int64_t m) {
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < m) x[i] += e[i];
}

// ---------------------------------------------------------------------------
// Cycle
// ---------------------------------------------------------------------------
static void ensure_vectors(lair_hierarchy *h, int32_t nrhs, hipStream_t s) {
    if (nrhs <= h->nrhs_cap) return;
    h->drop_graphs();     // captured iterations refer to the old buffers
    // a failed allocation below leaves no capacity claimed, so the next call
    // allocates every vector again
    h->nrhs_cap = 0;
    for_each_cycle_vector(h, nrhs, [&](auto &a, size_t count) { a.alloc(count, s); });
    h->partial.alloc((size_t)NPARTIAL * nrhs, s);
    h->norms.alloc((size_t)nrhs, s);
    h->nrhs_cap = nrhs;
}

// Algorithmic bytes of the cycle operations (w = value size, R = number of
// right-hand sides): every matrix entry (index + value), row pointer, source
// vector entry and destination entry counted once.
static double ab_rowdot(const DevCSR &M, int w, int R, int vec_in_out) {
    return (4.0 + w) * (double)M.nnz + 4.0 * (M.nrows + 1) + (double)w * R * M.ncols +
           (double)w * R * M.nrows * vec_in_out;
}
static double ab_jacobi(int64_t nnz_x, int32_t nx, int32_t n, int w, int R, bool sel) {
    return (4.0 + w) * (double)nnz_x + 12.0 * nx + (double)w * R * n + 2.0 * w * R * nx +
           (sel ? (double)n : 0.0);
}

template <class VT>
static void coarse_solve(lair_hierarchy *h, const VT *b, VT *x, int32_t nrhs,
                         bool transpose, hipStream_t s) {
    const int w = sizeof(VT);
    ProfScope ps("coarse_solve", s, 8.0 * h->coarse_entries + 2.0 * w * nrhs * h->nL,
                 2.0 * h->coarse_entries * nrhs);
    if (h->nsys > 1) {
        Level &Lb = *h->L.back();
        const uint8_t *act = h->use_act ? h->active_dev.get() : nullptr;
        auto block_solve = [&](const double *bb, double *xx) {
            if (h->binv.get())
                launch_block_apply_inv(h->nsys, Lb.seg_dev.get(), h->dense_off.get(),
                                       h->binv.get(), bb, xx, transpose, s, act,
                                       h->use_inv.get());
            launch_block_solve(h->nsys, Lb.seg_dev.get(), h->dense_off.get(), h->lu.get(),
                               h->piv.get(), bb, xx, transpose, s, act,
                               h->binv.get() ? h->use_inv.get() : nullptr);
        };
        if constexpr (std::is_same<VT, double>::value) {
            block_solve(b, x);
        } else {
            op_cast_f64(b, Lb.r.get(), h->nL, s);
            block_solve(Lb.r.get(), Lb.x.get());
            op_cast_f32(Lb.x.get(), x, h->nL, s);
        }
        return;
    }
    if (h->kinv.get()) {
        op_coarse_apply<VT>(h->nL, h->kinv.get(), b, x, nrhs, transpose, s);
        return;
    }
    Level &Lc = *h->L.back();
    if constexpr (std::is_same<VT, double>::value) {
        op_dense_solve<double>(h->nL, h->lu.get(), h->piv.get(), b, x, nrhs, transpose, s);
    } else {
        int64_t m = (int64_t)h->nL * nrhs;
        op_cast_f64(b, Lc.r.get(), m, s);
        op_dense_solve<double>(h->nL, h->lu.get(), h->piv.get(), Lc.r.get(), Lc.x.get(),
                               nrhs, transpose, s);
        op_cast_f32(Lc.x.get(), x, m, s);
    }
}

// F, F, C Jacobi sweeps on a level, every sweep reading the previous iterate.
// X is the iterate, Y a level-sized buffer:
//   F sweep 1 reads X, writes Y at the F rows;
//   F sweep 2 reads Y at F-points and X at C-points, writes X at the F rows
//     (X's F entries are not read by this sweep);
//   C sweep reads X, writes a compact buffer that is then scattered to X.
// With leave_c the C sweep writes Y's C rows instead and nothing is copied:
// the result is X at the F rows and Y at the C rows (on a split-ordered
// level, X below nf and Y from nf on).  Returns whether it did so.
template <class VT>
static bool ffc(lair_hierarchy *h, Level &Lv, const VT *b, VT *x, int32_t nrhs,
                hipStream_t s, bool leave_c) {
    const bool split = Lv.split;
    CsrView<VT> A = view<VT>(split ? Lv.As : Lv.A, Lv.team_A);
    if (nodal(h->opt)) {
        // block Jacobi x_X + D_X^{-1} (b - A x)_X is the scalar Jacobi sweep
        // on D^{-1} A (unit diagonal blocks) with right-hand side D^{-1} b
        VT *bt = vec<VT>(Lv.bt, Lv.bt32);
        {
            ProfScope ps("jacobi", s, 8.0 * Lv.n * h->opt.block_size +
                                          2.0 * sizeof(VT) * nrhs * Lv.n,
                         2.0 * Lv.n * h->opt.block_size * nrhs);
            op_node_rhs<VT>(Lv.n, h->opt.block_size, nrhs, Lv.ndinv.get(), b, bt, s);
        }
        b = bt;
        if constexpr (std::is_same<VT, double>::value) A.v = Lv.av.get();
        else A.v = Lv.av32.get();
    }
    VT *y = vec<VT>(Lv.t, Lv.t32);
    double om = h->opt.omega;
    const int w = sizeof(VT);
    // batch solve: only the rows of the systems still iterated (device lists)
    const bool act = h->use_act;
    // split ordering: F rows are 0 .. nf-1 and C rows nf .. n-1 (no list)
    const int32_t *frows = act ? Lv.act_f.get() : (split ? nullptr : Lv.flist.get());
    const int32_t *fcnt = act ? Lv.act_cnt + 1 : nullptr;
    if (act) {
        // the interpolation has written X and Y alike: F sweep 1 reads X and
        // writes Y's F rows, F sweep 2 reads Y and writes X's, and the C sweep
        // reads X at F-points and Y at C-points and writes X's C rows in place
        const int32_t ncr = Lv.nrc >= 0 ? Lv.nrc : Lv.nc;
        CsrView<VT> At = A;
        At.cjt = Lv.cjt.get();
        {
            ProfScope ps("jacobi", s, ab_jacobi(Lv.nnzF, Lv.nf, Lv.n, w, 1, false),
                         2.0 * Lv.nnzF);
            op_jacobi<VT>(A, frows, Lv.nf, b, x, x, nullptr, y, false, om, 1, s, fcnt);
        }
        {
            ProfScope ps("jacobi", s, ab_jacobi(Lv.nnzF, Lv.nf, Lv.n, w, 1, false),
                         2.0 * Lv.nnzF);
            op_jacobi<VT>(A, frows, Lv.nf, b, y, y, nullptr, x, false, om, 1, s, fcnt);
        }
        {
            ProfScope ps("jacobi", s, ab_jacobi(Lv.nnzC, ncr, Lv.n, w, 1, true),
                         2.0 * Lv.nnzC);
            op_jacobi<VT>(At, Lv.act_c.get(), ncr, b, x, y, Lv.cf.get(), x, false, om, 1, s,
                          Lv.act_cnt + 2);
        }
        return false;
    }
    {
        ProfScope ps("jacobi", s, ab_jacobi(Lv.nnzF, Lv.nf, Lv.n, w, nrhs, false),
                     2.0 * Lv.nnzF * nrhs);
        op_jacobi<VT>(A, frows, Lv.nf, b, x, x, nullptr, y, false, om, nrhs, s);
    }
    {
        ProfScope ps("jacobi", s, ab_jacobi(Lv.nnzF, Lv.nf, Lv.n, w, nrhs, true),
                     2.0 * Lv.nnzF * nrhs);
        CsrView<VT> At = A;
        At.cjt = split ? Lv.cjt_split.get() : Lv.cjt.get();
        op_jacobi<VT>(At, frows, Lv.nf, b, y, x, split ? Lv.cf_split.get() : Lv.cf.get(), x,
                      false, om, nrhs, s);
    }
    const int32_t *crows = split ? nullptr
                                 : (Lv.nrc >= 0 ? Lv.rclist.get() : Lv.clist.get());
    const int32_t ncr = Lv.nrc >= 0 ? Lv.nrc : Lv.nc;
    const int32_t c0 = split ? Lv.nf : 0;
    leave_c = leave_c && Lv.nrc < 0;
    {
        ProfScope ps("jacobi", s, ab_jacobi(Lv.nnzC, ncr, Lv.n, w, nrhs, false),
                     2.0 * Lv.nnzC * nrhs);
        op_jacobi<VT>(A, crows, ncr, b, x, x, nullptr, y, !leave_c, om, nrhs, s, nullptr, c0);
    }
    if (leave_c) return true;
    {
        ProfScope ps("scatter", s, 4.0 * ncr + 2.0 * w * nrhs * ncr);
        op_scatter<VT>(crows, ncr, y, x, nrhs, s, c0);
    }
    return false;
}

// ---------------------------------------------------------------------------
// The levels that one workgroup takes (k_tail.hip)
// ---------------------------------------------------------------------------
// A level is worth a workgroup while it is small: the workgroup moves its
// entries through one CU, the launches through the whole chip.  Solves of
// 2-D, 3-D and DG problems, microseconds per cycle in a graph (1, 4 and 16
// right-hand sides; "none": launches only), by the most entries a level of
// the tail may have:
//                            none   12,000  25,000  49,000
//   10^4 rows, distance 2      91      83      80      97
//   the same, 16 rhs          107      95      86      97
//   32^3 Euler                119     113     113     127
//   DG 32^2 x 2               124     118     118     124
//   DG 96^2 x 2               237     225     225     223
// The rows are bounded by what fits one CU's LDS in FP64; a float tail of
// more rows gained nothing (96^2 transport: 56 against 59 us).
constexpr int64_t TAIL_MAX_NNZ = 24576;
constexpr int32_t TAIL_MAX_ROWS = 4608;
constexpr int32_t TAIL_MAX_COARSE = 192;     // its inverse is read through one CU too
constexpr size_t TAIL_MAX_PACK = (size_t)256 << 20;
constexpr size_t TAIL_MAX_BATCH_PACK = (size_t)2 << 30;

// LDS of the tail from level t on with w-byte vectors, in bytes (see the
// kernels for what it holds).
static size_t tail_lds(const lair_hierarchy *h, size_t t, size_t w, bool transpose) {
    size_t e = 2 * ((size_t)h->L[t]->n + 1);
    if (!transpose) e += (size_t)h->L.back()->n + 1;
    else if (t + 1 < h->L.size()) e += (size_t)h->L[t + 1]->n + 1;
    for (size_t l = t; l < h->L.size(); ++l) e += (size_t)h->L[l]->n + 1;
    return e * w;
}

// First level of the tail of a single system (the number of levels: none).
static size_t tail_start(const lair_hierarchy *h, size_t w, bool transpose) {
    const size_t nl = h->L.size();
    if (h->nsys > 1 || !h->kinv.get() || h->nL > TAIL_MAX_COARSE) return nl;
    size_t t = nl;
    const size_t limit = std::min<size_t>(tail_lds_limit(), INT32_MAX);
    for (size_t l = nl - 1; l-- > 0;) {
        const Level &Lv = *h->L[l];
        if ((!transpose && Lv.split) || nl - l > (size_t)TAIL_MAX_LEVELS ||
            Lv.A.nnz > TAIL_MAX_NNZ || Lv.n > TAIL_MAX_ROWS || tail_lds(h, l, w, transpose) > limit)
            break;
        t = l;
    }
    return t;
}

template <class VT>
static const VT *values(const DevCSR &M) {
    if constexpr (std::is_same<VT, double>::value) return M.v.get();
    else return M.v32.get();
}

template <class VT>
static std::unique_ptr<TailArgs<VT>> &tail_args(Tail &t) {
    if constexpr (std::is_same<VT, double>::value) return t.a64;
    else return t.a32;
}

template <class VT>
static std::vector<TailSources<VT>> &tail_sources(Tail &t) {
    if constexpr (std::is_same<VT, double>::value) return t.src64;
    else return t.src32;
}

// Pack every level (again, when the operators have new values).
template <class VT>
static void pack_tail(Tail &t, hipStream_t s) {
    launch_tail_pack<VT>(tail_sources<VT>(t), s);
    t.stale = false;
}

static void repack(Tail &t, hipStream_t s) {
    if (!t.stale) return;
    if (t.w == 4) pack_tail<float>(t, s);
    else pack_tail<double>(t, s);
}

// Pack the tail's operators for nrhs right-hand sides (on s).
template <class VT>
static Tail make_tail(lair_hierarchy *h, size_t start, int32_t nrhs, bool transpose,
                      hipStream_t s) {
    Tail T;
    const int w = sizeof(VT);
    T.w = w;
    T.nrhs = nrhs;
    T.transpose = transpose;
    T.start = start;
    const size_t nl = h->L.size();
    const int32_t nlv = (int32_t)(nl - start);
    auto &a = tail_args<VT>(T);
    a.reset(new TailArgs<VT>());
    a->nlv = nlv;
    a->nrhs = nrhs;
    a->knode = nodal(h->opt) ? h->opt.block_size : 0;
    a->lds_bytes = (int32_t)tail_lds(h, start, w, transpose);
    a->omega = (VT)h->opt.omega;
    a->kinv = h->kinv.get();
    T.bytes = 8.0 * h->coarse_entries + 2.0 * w * nrhs * h->nL;
    T.flops = 2.0 * h->coarse_entries * nrhs;
    // longest rows: the transposes have to be measured
    std::vector<int32_t> longest(3 * (size_t)nlv, 0);
    if (transpose) {
        std::vector<const int32_t *> rp;
        std::vector<int32_t> n;
        for (int32_t k = 0; k + 1 < nlv; ++k) {
            Level &Lv = *h->L[start + k];
            for (const DevCSR *M : {&Lv.At, &Lv.Pt, &Lv.Rt}) {
                rp.push_back(M->rp.get());
                n.push_back(M->nrows);
            }
        }
        max_rows((int)rp.size(), rp.data(), n.data(), longest.data(), s);
    }
    auto &src = tail_sources<VT>(T);
    src.resize((size_t)nlv);
    size_t total = 0;
    for (int32_t k = 0; k < nlv; ++k) {
        Level &Lv = *h->L[start + k];
        TailLevel<VT> &o = a->lv[k];
        o.n = Lv.n;
        if (k + 1 == nlv) break;
        o.nf = Lv.nf;
        o.nc = Lv.nc;
        if (nodal(h->opt)) o.dinv = Lv.ndinv.get();
        const DevCSR &A = transpose ? Lv.At : Lv.A;
        const DevCSR &R = transpose ? Lv.Pt : Lv.R, &P = transpose ? Lv.Rt : Lv.P;
        const int32_t ta = transpose ? Lv.team_At : Lv.team_A;
        const int32_t la = transpose ? longest[3 * k] : Lv.max_row;
        const int32_t lr = transpose ? longest[3 * k + 1] : Lv.st.s_max + 1;
        // a row of P has one entry, or some of its row of A and itself
        const int32_t lp = transpose ? longest[3 * k + 2]
                           : h->opt.interp == LAIR_P_ONE_POINT ? 1 : Lv.max_row;
        for (int t = 0; t < TAIL_SETS; ++t) {
            TailSource<VT> &S = src[k].src[t];
            // the residual of every row: the transposed cycle's, and that of
            // an iterate given to the first level
            if (t == TAIL_A && !transpose && (w == 4 || k > 0 || start > 0)) continue;
            const DevCSR &M = t == TAIL_R ? R : t == TAIL_P ? P : A;
            const int32_t len = t == TAIL_R ? lr : t == TAIL_P ? lp : la;
            const int32_t team = t == TAIL_R ? (transpose ? Lv.team_Pt : Lv.team_R)
                                 : t == TAIL_P ? (transpose ? Lv.team_Rt : Lv.team_P) : ta;
            S.rp = M.rp.get();
            S.cj = M.cj.get();
            S.v = values<VT>(M);
            const bool sweep = t == TAIL_F || t == TAIL_C;
            if (sweep && nodal(h->opt)) S.v = vec<VT>(Lv.av, Lv.av32);
            S.rows = t == TAIL_F ? Lv.flist.get() : t == TAIL_C ? Lv.clist.get() : nullptr;
            S.n = t == TAIL_F ? Lv.nf : t == TAIL_C ? Lv.nc : M.nrows;
            S.ncol = M.ncols;
            S.diag = sweep;
            cycle_team(team, nrhs, w, sweep, &S.lg, &S.ll);
            S.nchunk = tail_chunks(S.n, S.lg);
            S.dst.lg = S.lg;
            // one entry a lane: one-point interpolation
            S.dst.u4 = t != TAIL_P || tail_groups(len, S.lg, S.ll, false) > 1;
            const int32_t g = tail_groups(len, S.lg, S.ll, S.dst.u4);
            if (g > UINT16_MAX) return Tail();
            S.dst.smax = (uint16_t)g;
            total = tail_layout(S.dst, total, S.nchunk, sweep, w);
        }
        T.bytes += ab_rowdot(Lv.R, w, nrhs, 1) + ab_rowdot(Lv.P, w, nrhs, 1) +
                   2.0 * ab_jacobi(Lv.nnzF, Lv.nf, Lv.n, w, nrhs, false) +
                   ab_jacobi(Lv.nnzC, Lv.nc, Lv.n, w, nrhs, false) +
                   (transpose ? ab_rowdot(Lv.A, w, nrhs, 2) : 0.0);
        T.flops += 2.0 * nrhs * ((double)Lv.R.nnz + Lv.P.nnz + 2.0 * Lv.nnzF + Lv.nnzC +
                                 (transpose ? Lv.A.nnz : 0));
    }
    if (total > TAIL_MAX_PACK) return Tail();
    T.blob.alloc(std::max<size_t>(total, 256), s);
    a->blob = T.blob.get();
    for (int32_t k = 0; k + 1 < nlv; ++k) {
        src[k].blob = T.blob.get();
        for (int t = 0; t < TAIL_SETS; ++t) a->lv[k].set[t] = src[k].src[t].dst;
    }
    pack_tail<VT>(T, s);
    return T;
}

// The tail a cycle of this kind uses from level l on, or nullptr (one packed
// from old values is not used).
template <class VT>
static Tail *find_tail(lair_hierarchy *h, int32_t nrhs, bool transpose, size_t l) {
    for (auto &t : h->tails)
        if (t.w == (int)sizeof(VT) && t.nrhs == nrhs && t.transpose == transpose)
            return l >= t.start && tail_args<VT>(t) && !t.stale ? &t : nullptr;
    return nullptr;
}

// What make() returns, or nothing when there is no memory for it: the cycle
// runs without a tail, so a call that fits without one does not fail for it.
template <class Make>
static auto unless_no_memory(Make &&make) -> decltype(make()) {
    try {
        return make();
    } catch (const Error &e) {
        if (e.status != LAIR_ENOMEM) throw;
        return {};
    }
}

// Work queued on s would only be recorded (also when that cannot be told).
static bool capturing(hipStream_t s) {
    hipStreamCaptureStatus cs = hipStreamCaptureStatusNone;
    if (hipStreamIsCapturing(s, &cs) == hipSuccess && cs == hipStreamCaptureStatusNone) return false;
    (void)hipGetLastError();
    return true;
}

// Make the tail of a cycle kind, or pack it again after new values.  Not while
// the stream is captured: the cycle then runs launch by launch, the same sums.
static void ensure_tail(lair_hierarchy *h, int32_t nrhs, bool mixed, bool transpose,
                        hipStream_t s) {
    const int w = mixed ? 4 : 8;
    Tail *have = nullptr;
    for (auto &t : h->tails)
        if (t.w == w && t.nrhs == nrhs && t.transpose == transpose) have = &t;
    if (have && !have->stale) return;
    if (capturing(s)) return;
    if (have) {
        repack(*have, s);
        return;
    }
    const size_t start = tail_start(h, w, transpose);
    Tail T;
    if (start < h->L.size())
        T = unless_no_memory([&] {
            return mixed ? make_tail<float>(h, start, nrhs, transpose, s)
                         : make_tail<double>(h, start, nrhs, transpose, s);
        });
    T.w = w;
    T.nrhs = nrhs;
    T.transpose = transpose;
    h->drop_graphs();        // captured without it
    h->tails.push_back(std::move(T));
}

// Whether tails are worth their workgroups on a batch.  Up to one system a CU
// (a workgroup's 1,024 threads take its registers) all of them take as long as
// the largest; beyond, each level of a system costs a CU about 9.5 us.  A
// launched level costs 21 us and the coarsest solve 8, and the rows 1 us per
// 4,500.  Microseconds per iteration (30 iterations, m x m grids):
//   levels   m     systems: tails / launches
//     1     11      300:  58 /  67    1,000:  87 /  76
//     2     13      500:  68 /  83    1,500: 133 / 103    2,000: 168 / 118
//     3     16    1,000: 112 / 125    2,000: 212 / 171
//     4     24    1,000: 171 / 200    2,000: 311 / 331
//     6     40      128:  76 / 171    1,000: 276 / 421
//     7     66      300: 251 / 408
static bool batch_tail_pays(const lair_hierarchy *h, const Tail &T) {
    int dev = 0, cus = 0;
    LAIR_HIP(hipGetDevice(&dev));
    LAIR_HIP(hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev));
    double levels = 0.0, rows = 0.0;
    for (int32_t q = 0; q < h->nsys; ++q) {
        const Level &Lv = *h->L[T.top[q]];
        levels += h->sys_levels[q] - T.top[q];
        rows += (double)(Lv.seg[q + 1] - Lv.seg[q]);
    }
    return 9.5 * levels / std::max(1, cus) <=
           8.0 + 21.0 * (double)(h->L.size() - 1 - T.start) + rows / 4500.0;
}

// The tail of a batch solve: one workgroup per system, from the first level
// at which the system is as small as a single system's tail may be (its
// entries taken from the union's mean row).  Systems of a batch differ by a
// factor of a hundred, so each has a start of its own; the levels above are
// launched over the systems that still need them, and the tail is launched
// where the last system's starts.  nullptr: no tail (a coarsest block without
// an inverse, too many levels, or systems for which it does not pay).
template <class VT>
static std::unique_ptr<Tail> make_batch_tail(lair_hierarchy *h,
                                             const std::vector<std::array<std::vector<int32_t>, 3>> &runs,
                                             hipStream_t s) {
    const int w = sizeof(VT);
    const int32_t ns = h->nsys, nl = (int32_t)h->L.size();
    const std::vector<int64_t> &cs = h->L.back()->seg;
    if (nl > TAIL_MAX_LEVELS || !h->binv.get()) return nullptr;
    for (int32_t q = 0; q < ns; ++q)
        if (cs[q + 1] - cs[q] > mid_dense_max()) return nullptr;
    auto rows = [&](int32_t l, int32_t q) {
        return (int64_t)(h->L[l]->seg[q + 1] - h->L[l]->seg[q]);
    };
    std::unique_ptr<Tail> T(new Tail());
    T->w = w;
    T->nrhs = 1;
    T->top.assign((size_t)ns, 0);
    const size_t limit = std::min<size_t>(tail_lds_limit(), INT32_MAX);
    size_t lds = 0;
    int32_t depth = 0;
    for (int32_t q = 0; q < ns; ++q) {
        const int32_t last = h->sys_levels[q] - 1;
        size_t below = 2 * ((size_t)rows(last, q) + 1);     // coarsest vectors
        int32_t t = last;
        for (int32_t l = last - 1; l >= 0; --l) {
            const int64_t n = rows(l, q);
            const double mean = (double)h->L[l]->A.nnz / std::max(h->L[l]->n, 1);
            below += (size_t)n + 1;
            if (n > TAIL_MAX_ROWS || n * mean > (double)TAIL_MAX_NNZ ||
                (below + 2 * ((size_t)n + 1)) * w > limit)
                break;
            t = l;
        }
        size_t e = 2 * ((size_t)rows(t, q) + 1) + (size_t)rows(last, q) + 1;
        for (int32_t l = t; l <= last; ++l) e += (size_t)rows(l, q) + 1;
        if (e * w > limit) return nullptr;
        lds = std::max(lds, e * w);
        T->top[q] = t;
        depth = std::max(depth, t);
    }
    T->start = (size_t)depth;
    if (!batch_tail_pays(h, *T)) return nullptr;
    auto &a = tail_args<VT>(*T);
    a.reset(new TailArgs<VT>());
    a->nlv = nl;
    a->nrhs = 1;
    a->nsys = ns;
    a->lds_bytes = (int32_t)lds;
    a->omega = (VT)h->opt.omega;
    a->doff = h->dense_off.get();
    a->binv = h->binv.get();
    a->active = h->active_dev.get();
    // tables: order, top, levels, then per level the F and C runs and the
    // first chunks of every set
    const size_t per = (size_t)ns + 1, lvt = (2 + TAIL_SETS) * per;
    std::vector<int32_t> tab(3 * (size_t)ns + lvt * (size_t)nl, 0);
    std::vector<int32_t> order((size_t)ns);
    for (int32_t q = 0; q < ns; ++q) order[q] = q;
    std::stable_sort(order.begin(), order.end(), [&](int32_t x, int32_t y) {
        return rows(T->top[x], x) > rows(T->top[y], y);
    });
    std::copy(order.begin(), order.end(), tab.begin());
    std::copy(T->top.begin(), T->top.end(), tab.begin() + ns);
    std::copy(h->sys_levels.begin(), h->sys_levels.end(), tab.begin() + 2 * ns);
    T->tables.alloc(tab.size(), s);
    const int32_t *d = T->tables.get();
    a->order = d;
    a->top = d + ns;
    a->slev = d + 2 * ns;
    T->bytes = 8.0 * h->coarse_entries + 2.0 * w * h->nL;
    T->flops = 2.0 * h->coarse_entries;
    auto &src = tail_sources<VT>(*T);
    src.resize((size_t)nl);
    size_t total = 0;
    for (int32_t l = 0; l < nl; ++l) {
        Level &Lv = *h->L[l];
        TailLevel<VT> &o = a->lv[l];
        o.n = Lv.n;
        o.seg = Lv.seg_dev.get();
        if (l + 1 == nl) break;
        Level &Nx = *h->L[l + 1];
        o.nf = Lv.nf;
        o.nc = Lv.nrc >= 0 ? Lv.nrc : Lv.nc;
        int32_t *t0 = tab.data() + 3 * ns + lvt * l;
        const int32_t *d0 = d + 3 * ns + lvt * l;
        std::copy(runs[l][1].begin(), runs[l][1].end(), t0);
        std::copy(runs[l][2].begin(), runs[l][2].end(), t0 + per);
        o.frun = d0;
        o.crun = d0 + per;
        o.chunk0 = d0 + 2 * per;
        for (int t = 0; t < TAIL_A; ++t) {
            TailSource<VT> &S = src[l].src[t];
            const DevCSR &M = t == TAIL_R ? Lv.R : t == TAIL_P ? Lv.P : Lv.A;
            const int32_t len = t == TAIL_R ? Lv.st.s_max + 1
                                : t == TAIL_P && h->opt.interp == LAIR_P_ONE_POINT ? 1
                                                                                  : Lv.max_row;
            const bool sweep = t == TAIL_F || t == TAIL_C;
            S.rp = M.rp.get();
            S.cj = M.cj.get();
            S.v = values<VT>(M);
            S.rows = t == TAIL_F ? Lv.flist.get()
                     : t == TAIL_C ? (Lv.nrc >= 0 ? Lv.rclist.get() : Lv.clist.get()) : nullptr;
            S.run = t == TAIL_F ? o.frun : o.crun;
            S.rseg = t == TAIL_R ? Nx.seg_dev.get() : Lv.seg_dev.get();
            S.cseg = t == TAIL_P ? Nx.seg_dev.get() : Lv.seg_dev.get();
            S.chunk0 = o.chunk0 + t * per;
            S.nsys = ns;
            S.diag = sweep;
            cycle_team(t == TAIL_R ? Lv.team_R : t == TAIL_P ? Lv.team_P : Lv.team_A, 1, w,
                       sweep, &S.lg, &S.ll);
            S.dst.lg = S.lg;
            S.dst.u4 = t != TAIL_P || tail_groups(len, S.lg, S.ll, false) > 1;
            const int32_t g = tail_groups(len, S.lg, S.ll, S.dst.u4);
            if (g > UINT16_MAX) return nullptr;
            S.dst.smax = (uint16_t)g;
            int32_t *c0 = t0 + (2 + t) * per;
            for (int32_t q = 0; q < ns; ++q) {
                int32_t n = 0;
                if (l >= T->top[q] && l + 1 < h->sys_levels[q])
                    n = t == TAIL_R ? (int32_t)rows(l + 1, q) : t == TAIL_P ? (int32_t)rows(l, q)
                        : runs[l][t == TAIL_F ? 1 : 2][q + 1] - runs[l][t == TAIL_F ? 1 : 2][q];
                c0[q + 1] = c0[q] + tail_chunks(n, S.lg);
            }
            S.nchunk = c0[ns];
            total = tail_layout(S.dst, total, S.nchunk, sweep, w);
        }
        double share = 0.0;
        for (int32_t q = 0; q < ns; ++q)
            if (l >= T->top[q] && l + 1 < h->sys_levels[q]) share += (double)rows(l, q);
        share /= std::max(Lv.n, 1);
        T->bytes += share * (ab_rowdot(Lv.R, w, 1, 1) + ab_rowdot(Lv.P, w, 1, 1) +
                             2.0 * ab_jacobi(Lv.nnzF, Lv.nf, Lv.n, w, 1, false) +
                             ab_jacobi(Lv.nnzC, o.nc, Lv.n, w, 1, false));
        T->flops += share * 2.0 * ((double)Lv.R.nnz + Lv.P.nnz + 2.0 * Lv.nnzF + Lv.nnzC);
    }
    if (total > TAIL_MAX_BATCH_PACK) return nullptr;
    T->blob.alloc(std::max<size_t>(total, 256), s);
    int32_t *st = (int32_t *)pinned_upload(sizeof(int32_t) * tab.size());
    memcpy(st, tab.data(), sizeof(int32_t) * tab.size());
    LAIR_HIP(hipMemcpyAsync(T->tables.get(), st, sizeof(int32_t) * tab.size(),
                            hipMemcpyHostToDevice, s));
    a->blob = T->blob.get();
    for (int32_t l = 0; l + 1 < nl; ++l) {
        src[l].blob = T->blob.get();
        for (int t = 0; t < TAIL_A; ++t) a->lv[l].set[t] = src[l].src[t].dst;
    }
    pack_tail<VT>(*T, s);
    LAIR_HIP(hipStreamSynchronize(s));     // the staging area is reused
    return T;
}

// V-cycle from level l.  With x_zero the incoming iterate is zero: the
// residual is b itself and the interpolated correction is assigned.  When
// r is non-null it already holds b - A x.  With split_out the result may be
// left split (see ffc): the return value is then the buffer that holds its
// C rows, otherwise nullptr (x holds all of it).
template <class VT>
static const VT *vcycle(lair_hierarchy *h, size_t l, const VT *b, VT *x, bool x_zero,
                        const VT *r, int32_t nrhs, hipStream_t s, bool split_out = false) {
    Level &Lv = *h->L[l];
    const int w = sizeof(VT);
    if (h->use_act && h->batch_tail && l == h->batch_tail->start) {
        Tail &T = *h->batch_tail;
        ProfScope ps("tail", s, T.bytes, T.flops);
        launch_tail<VT>(*tail_args<VT>(T), TAIL_ZERO, nullptr, nullptr, nullptr, s);
        return nullptr;
    }
    if (l + 1 == h->L.size()) {
        coarse_solve<VT>(h, b, x, nrhs, false, s);
        return nullptr;
    }
    if (Tail *T = h->use_act ? nullptr : find_tail<VT>(h, nrhs, false, l)) {
        ProfScope ps("tail", s, T->bytes, T->flops);
        launch_tail<VT>(*tail_args<VT>(*T), x_zero ? TAIL_ZERO : r ? TAIL_RESID : TAIL_ITERATE,
                        b, x, r, s);
        return nullptr;
    }
    Level &Nx = *h->L[l + 1];
    const VT *res = b;
    if (!x_zero) {
        if (r) {
            res = r;
        } else {
            VT *rr = vec<VT>(Lv.r, Lv.r32);
            ProfScope ps("residual", s, ab_rowdot(Lv.A, w, nrhs, 2), 2.0 * Lv.A.nnz * nrhs);
            op_residual<VT>(view<VT>(Lv.split ? Lv.As : Lv.A, Lv.team_A), b, x, rr, nrhs, s);
            res = rr;
        }
    }
    VT *bc = vec<VT>(Nx.b, Nx.b32);
    VT *xc = vec<VT>(Nx.x, Nx.x32);
    {
        ProfScope ps("restrict", s, ab_rowdot(Lv.R, w, nrhs, 1), 2.0 * Lv.R.nnz * nrhs);
        if (h->use_act)
            op_rowdot_list<VT>(view<VT>(Lv.R, Lv.team_R), 1, Nx.act_rows.get(),
                               Nx.act_cnt, Nx.n, res, nullptr, bc, s);
        else
            op_spmv<VT>(view<VT>(Lv.Rs.rp.get() ? Lv.Rs : Lv.R, Lv.team_R), res, bc, nrhs, false,
                        s);
    }
    // the coarse correction may come back in two buffers (its C rows in the
    // level's work buffer); the interpolation then reads those columns there
    const bool coarse_split = !h->use_act &&
                              op_spmv_split_ok(nrhs, xc, vec<VT>(Nx.t, Nx.t32), x);
    const VT *xc_hi = vcycle<VT>(h, l + 1, bc, xc, true, nullptr, nrhs, s, coarse_split);
    {
        ProfScope ps("interpolate", s, ab_rowdot(Lv.P, w, nrhs, x_zero ? 1 : 2),
                     2.0 * Lv.P.nnz * nrhs);
        if (h->use_act)
            op_rowdot_list<VT>(view<VT>(Lv.P, Lv.team_P), x_zero ? 1 : 2, Lv.act_p.get(),
                               Lv.act_cnt + 3, Lv.n, xc, nullptr, x, s,
                               vec<VT>(Lv.t, Lv.t32));
        else
            op_spmv<VT>(view<VT>(Lv.Ps.rp.get() ? Lv.Ps : Lv.P, Lv.team_P), xc, x, nrhs, !x_zero,
                        s, xc_hi, Nx.split && nrhs > 1 ? Nx.nf : -1,
                        Nx.split ? Nx.cf_split.get() : Nx.cf.get());
    }
    return ffc<VT>(h, Lv, b, x, nrhs, s, split_out) ? vec<VT>(Lv.t, Lv.t32) : nullptr;
}

// Transposed cycle: C, F, F Jacobi on A^T, restriction with P^T, recursion
// on K^T, interpolation with R^T.
static void ensure_transposes(lair_hierarchy *h, hipStream_t cs) {
    if (h->have_transpose && !h->transpose_stale) return;
    const size_t nl = h->L.size();
    if (h->have_transpose) {
        // new values on the kept patterns; under capture at once, on the
        // stream of the new diagonal: recorded, they would be missing from
        // every call before the graph's first replay
        const bool aside = capturing(cs);
        if (aside) {
            cs = h->stream;
            if (capturing(cs))
                fail(LAIR_EDEVICE, "the transposed operators of a new diagonal cannot be made "
                     "while its stream is captured");
        }
        TransposeValues t{};
        int m = 0;
        auto add = [&](const DevCSR &M, DevCSR &T, const DevArr<int32_t> &pos) {
            t.m[m++] = {M.v.get(), pos.get(), T.v.get(), M.nnz};
            if (m == 96) {
                launch_transpose_values(t, m, cs);
                m = 0;
            }
        };
        for (size_t l = 0; l < nl; ++l) {
            Level &Lv = *h->L[l];
            add(Lv.A, Lv.At, Lv.At_pos);
            if (l + 1 == nl) break;
            add(Lv.R, Lv.Rt, Lv.Rt_pos);
            add(Lv.P, Lv.Pt, Lv.Pt_pos);
            launch_diagonal(Lv.n, Lv.A.rp.get(), Lv.A.cj.get(), Lv.A.v.get(), Lv.tdiag.get(), cs);
        }
        if (m) launch_transpose_values(t, m, cs);
        if (aside) LAIR_HIP(hipStreamSynchronize(cs));
        h->transpose_stale = false;
        return;
    }
    hipStream_t s = h->stream;
    DevArr<int64_t> tmp;
    for (size_t l = 0; l < nl; ++l) {
        Level &Lv = *h->L[l];
        transpose(Lv.A, Lv.At, Lv.At_pos, s, tmp);
        Lv.team_At = team_of(Lv.At);
        if (l + 1 == nl) break;
        transpose(Lv.R, Lv.Rt, Lv.Rt_pos, s, tmp);
        transpose(Lv.P, Lv.Pt, Lv.Pt_pos, s, tmp);
        Lv.team_Rt = team_of(Lv.Rt);
        Lv.team_Pt = team_of(Lv.Pt);
        Lv.tdiag.alloc((size_t)std::max(Lv.n, 1), s);
        launch_diagonal(Lv.n, Lv.A.rp.get(), Lv.A.cj.get(), Lv.A.v.get(), Lv.tdiag.get(), s);
        Lv.tkind.alloc((size_t)std::max(Lv.n, 1), s);
        launch_row_kind(Lv.n, Lv.nrc >= 0 ? Lv.rclist.get() : Lv.clist.get(),
                        Lv.nrc >= 0 ? Lv.nrc : Lv.nc, Lv.tkind.get(), s);
    }
    LAIR_HIP(hipStreamSynchronize(s));
    h->have_transpose = true;
    h->transpose_stale = false;
}

// lam = B^T g from zero.  The C sweep of a zero iterate writes lam and the
// work vector t; the first F sweep reads lam and writes t's F rows, the second
// reads t and writes lam's.
static void vcycle_t(lair_hierarchy *h, size_t l, const double *g, double *lam, int32_t nrhs,
                     hipStream_t s) {
    Level &Lv = *h->L[l];
    if (l + 1 == h->L.size()) {
        coarse_solve<double>(h, g, lam, nrhs, true, s);
        return;
    }
    if (Tail *T = find_tail<double>(h, nrhs, true, l)) {
        ProfScope ps("tail", s, T->bytes, T->flops);
        launch_tail_t(*T->a64, g, lam, s);
        return;
    }
    CsrView<double> At = view<double>(Lv.At, Lv.team_At);
    const double om = h->opt.omega;
    double *t = Lv.t.get();
    op_first_sweep(Lv.n, nrhs, Lv.tkind.get(), g, Lv.tdiag.get(), om, lam, t, s);
    op_jacobi<double>(At, Lv.flist.get(), Lv.nf, g, lam, lam, nullptr, t, false, om, nrhs, s);
    op_jacobi<double>(At, Lv.flist.get(), Lv.nf, g, t, t, nullptr, lam, false, om, nrhs, s);
    op_residual<double>(At, g, lam, Lv.r.get(), nrhs, s);
    Level &Nx = *h->L[l + 1];
    op_spmv<double>(view<double>(Lv.Pt, Lv.team_Pt), Lv.r.get(), Nx.b.get(), nrhs, false, s);
    vcycle_t(h, l + 1, Nx.b.get(), Nx.x.get(), nrhs, s);
    op_spmv<double>(view<double>(Lv.Rt, Lv.team_Rt), Nx.x.get(), lam, nrhs, true, s);
}

static bool valid_nrhs(int32_t nrhs) {
    return nrhs == 1 || nrhs == 2 || nrhs == 4 || nrhs == 8 || nrhs == 16 || nrhs == 32;
}

// After a new diagonal that failed the levels hold values of both diagonals
// and the coarsest grid may have neither an inverse nor factors (its pivots
// are then whatever the memory held).
static void check_usable(const lair_hierarchy *h) {
    if (!h->usable)
        fail(LAIR_EINVAL, "the last new diagonal failed: the hierarchy is unusable until an "
             "update succeeds");
}

void check_nrhs(const lair_hierarchy *h, int32_t nrhs) {
    check_usable(h);
    if (!valid_nrhs(nrhs)) fail(LAIR_EINVAL, "nrhs must be 1, 2, 4, 8, 16 or 32");
    if (h->nsys > 1 && nrhs != 1)
        fail(LAIR_EINVAL, "a hierarchy of a batch takes one right-hand side per system");
}

static void sumsq_dev(lair_hierarchy *h, const double *r, int32_t nrhs, hipStream_t s) {
    ProfScope ps("norm", s, 8.0 * nrhs * h->L[0]->n, 2.0 * nrhs * h->L[0]->n);
    op_sumsq(r, h->L[0]->n, nrhs, h->partial.get(), NPARTIAL, h->norms.get(), s);
}

// Square roots of the m sums of squares at dev (synchronises s).
static void read_norms(const double *dev, int32_t m, hipStream_t s, std::vector<double> &out) {
    out.resize((size_t)m);
    {
        Readback rb(s);
        rb.add(out.data(), dev, sizeof(double) * m);
        rb.run();
    }
    for (auto &v : out) v = std::sqrt(v);
}

static void norms_host(lair_hierarchy *h, const double *r, int32_t nrhs,
                       hipStream_t s, std::vector<double> &out) {
    sumsq_dev(h, r, nrhs, s);
    read_norms(h->norms.get(), nrhs, s, out);
}

// Kinds of captured iterations.
enum { IT_FP64 = 0, IT_MIXED = 1, IT_BATCH_FP64 = 2, IT_BATCH_MIXED = 3, IT_TRANSPOSE = 4 };

static const char *const CYCLE_CATEGORIES[] = {
    "jacobi", "scatter", "residual", "restrict", "interpolate", "coarse_solve", "norm", "cast",
    "tail"};

// Iterations are captured unless the caller asked for eager launches or the
// profiler times one of the cycle's categories (its events would have to be
// recorded launch by launch).
static bool use_graphs(const lair_hierarchy *h) {
    if (h->opt.flags & LAIR_FLAG_NO_GRAPH) return false;
    for (const char *c : CYCLE_CATEGORIES)
        if (prof_selected(c)) return false;
    return true;
}

static const size_t MAX_GRAPHS = 8;

// Iterations of a kind launched before it is captured.  Capturing and
// instantiating costs the host 0.1 to 0.4 ms, a replay saves a few
// microseconds over launching what the tail leaves of a cycle (97 x 97, 17
// iterations: 1.91 ms captured at once, 1.83 launched, 1.53 replayed; 80^3,
// 10 iterations: 3.39, 3.23, 2.93), so a graph pays for combinations that
// keep coming back.
static const int GRAPH_AFTER = 24;

// Run body(stream) on s.  The first iterations of a kind are launched
// directly; then one is captured on the hierarchy's private stream, and later
// ones replay its graph.  body must launch kernels only (no allocation, no
// host synchronisation, no memset).
template <class Body>
static void run_iteration(lair_hierarchy *h, int kind, int32_t nrhs, const void *b, void *x,
                          hipStream_t s, Body &&body) {
    if (!use_graphs(h)) {
        body(s);
        return;
    }
    lair_hierarchy::Graph *g = nullptr;
    for (auto &k : h->graphs)
        if (k.kind == kind && k.nrhs == nrhs && k.b == b && k.x == x) g = &k;
    if (!g) {
        if (h->graphs.size() >= MAX_GRAPHS) {
            if (h->graphs.front().exec) (void)hipGraphExecDestroy(h->graphs.front().exec);
            h->graphs.erase(h->graphs.begin());
        }
        h->graphs.push_back({kind, nrhs, b, x, 0, nullptr});
        g = &h->graphs.back();
    }
    if (g->exec) {
        ProfScope ps("graph", s, 0.0);
        hipEvent_t e0 = nullptr, e1 = nullptr;
        const bool timed = prof_kernel_events(s, &e0, &e1);
        if (timed) LAIR_HIP(hipEventRecord(e0, s));
        LAIR_HIP(hipGraphLaunch(g->exec, s));
        if (timed) LAIR_HIP(hipEventRecord(e1, s));
        return;
    }
    body(s);
    if (++g->runs < GRAPH_AFTER) return;
    if (!h->gstream) LAIR_HIP(hipStreamCreateWithFlags(&h->gstream, hipStreamNonBlocking));
    hipGraph_t graph = nullptr;
    LAIR_HIP(hipStreamBeginCapture(h->gstream, hipStreamCaptureModeThreadLocal));
    try {
        body(h->gstream);
    } catch (...) {
        if (hipStreamEndCapture(h->gstream, &graph) == hipSuccess && graph)
            (void)hipGraphDestroy(graph);
        throw;
    }
    LAIR_HIP(hipStreamEndCapture(h->gstream, &graph));
    hipGraphExec_t exec = nullptr;
    hipError_t e = hipGraphInstantiate(&exec, graph, nullptr, nullptr, 0);
    (void)hipGraphDestroy(graph);
    if (e != hipSuccess) fail(LAIR_EDEVICE, "graph instantiation failed: %s", hipGetErrorString(e));
    g->exec = exec;
}

static void check_solve_args(lair_hierarchy *h, const double *b, double *x, double rtol,
                             int32_t maxit) {
    if (!h) fail(LAIR_EINVAL, "hierarchy is NULL");
    if (!b || !x) fail(LAIR_EINVAL, "b and x must not be NULL");
    if (!(rtol > 0.0) || maxit < 0) fail(LAIR_EINVAL, "need rtol > 0 and maxit >= 0");
}

void info_common(const lair_hierarchy *h, lair_info *info) {
    info->nlevels = (int32_t)h->L.size();
    info->cycle_complexity = h->cc;
    info->op_complexity = h->oc;
    info->n_singular_local = h->n_singular;
    info->setup_ms = h->setup_ms;
    info->split_ms = h->split_ms;
    for (int k = 0; k < 8; ++k) info->setup_phase_ms[k] = h->phase_ms[k];
    // Sec. 4: work units per digit of accuracy, -CC / log10(rho)
    info->wpd = (info->rho > 0.0 && info->rho < 1.0)
                    ? -h->cc / std::log10(info->rho) : 0.0;
    info->hist_len = 0;
}

static void set_history(lair_info *info, const std::vector<double> &hist) {
    const size_t m = std::min(hist.size(), (size_t)LAIR_HIST_MAX);
    for (size_t k = 0; k < m; ++k) info->relres_hist[k] = hist[k];
    info->hist_len = (int32_t)m;
}

lair_status solve_impl(lair_hierarchy *h, const double *b, double *x,
                       int32_t nrhs, double rtol, int32_t maxit,
                       lair_info *info, hipStream_t s, bool transpose) {
    auto t0 = Clock::now();
    check_solve_args(h, b, x, rtol, maxit);
    check_nrhs(h, nrhs);
    ensure_vectors(h, nrhs, s);
    if (transpose) ensure_transposes(h, s);
    ensure_tail(h, nrhs, h->opt.precision == LAIR_MIXED && !transpose, transpose, s);
    Level &L0 = *h->L[0];
    const int64_t n = L0.n;
    const double *bb = b;
    if (scaled(h->opt) && !transpose) {
        op_block_apply(n / h->opt.block_size, h->opt.block_size, h->dinv.get(), b,
                       h->bscaled.get(), nrhs, s);
        bb = h->bscaled.get();
    }
    bool mixed = h->opt.precision == LAIR_MIXED && !transpose;
    // level 0 renumbered for the cycle: the FP64 iteration carries b and x
    // in the split ordering (x is written back at the end); the mixed one
    // keeps them natural, writes its float residual in the split ordering
    // and adds the correction back row by row
    const bool split = L0.split && !transpose;
    const bool vec_split = split && !mixed;
    const int32_t *orow = split && mixed ? L0.iperm.get() : nullptr;
    double *const xu = x;
    if (vec_split) {
        op_permute_rows(n, nrhs, L0.perm.get(), bb, h->bsplit.get(), true, s);
        op_permute_rows(n, nrhs, L0.perm.get(), x, h->xsplit.get(), true, s);
        bb = h->bsplit.get();
        x = h->xsplit.get();
    }
    std::vector<double> nb, rn, r_first;
    norms_host(h, bb, nrhs, s, nb);
    CsrView<double> A0 = transpose ? view<double>(L0.At, L0.team_At)
                                   : view<double>(vec_split ? L0.As : L0.A, L0.team_A);
    const DevCSR &M0 = transpose ? L0.At : L0.A;
    // fused residual + norms (+ float copy in mixed precision) unless the
    // caller's vectors are not 16-byte aligned
    const bool fused = nrhs == 1 || (((uintptr_t)bb | (uintptr_t)x) & 15u) == 0;
    auto residual_and_norms = [&](hipStream_t st) {
        if (fused) {
            ProfScope ps("residual", st, ab_rowdot(M0, 8, nrhs, 1) + (mixed ? 4.0 : 8.0) *
                         nrhs * (double)M0.nrows, 2.0 * M0.nnz * nrhs);
            if (!op_residual_norm(A0, bb, x, mixed ? nullptr : h->r0.get(),
                                  mixed ? h->r0_32.get() : nullptr, nrhs, h->partial.get(),
                                  NPARTIAL, h->norms.get(), st, orow))
                fail(LAIR_EDEVICE, "fused residual not applicable");
            return;
        }
        {
            ProfScope ps("residual", st, ab_rowdot(M0, 8, nrhs, 2), 2.0 * M0.nnz * nrhs);
            op_residual<double>(A0, bb, x, h->r0.get(), nrhs, st);
        }
        sumsq_dev(h, h->r0.get(), nrhs, st);
    };
    residual_and_norms(s);
    read_norms(h->norms.get(), nrhs, s, rn);
    r_first = rn;
    int32_t it = 0;
    double relmax = 0.0;
    std::vector<double> hist;
    for (;;) {
        relmax = 0.0;
        bool done = true;
        for (int32_t q = 0; q < nrhs; ++q) {
            double rel = nb[q] > 0 ? rn[q] / nb[q] : rn[q];
            relmax = std::max(relmax, rel);
            if (!(rel <= rtol)) done = false;
        }
        hist.push_back(relmax);
        if (done || it >= maxit) break;
        if (transpose) {
            // lambda <- lambda + B^T (g - A^T lambda): cycle on the residual
            run_iteration(h, IT_TRANSPOSE, nrhs, bb, x, s, [&](hipStream_t st) {
                vcycle_t(h, 0, h->r0.get(), L0.b.get(), nrhs, st);
                LAIR_LAUNCH(k_add, dim3(blocks_for(n * nrhs, 256)), dim3(256), 0, st, x,
                            L0.b.get(), n * nrhs);
                LAIR_LAUNCH_CHECK();
                residual_and_norms(st);
            });
        } else if (!mixed) {
            run_iteration(h, IT_FP64, nrhs, bb, x, s, [&](hipStream_t st) {
                vcycle<double>(h, 0, bb, x, false, h->r0.get(), nrhs, st);
                residual_and_norms(st);
            });
        } else {
            run_iteration(h, IT_MIXED, nrhs, bb, x, s, [&](hipStream_t st) {
                if (!fused) {
                    ProfScope ps("cast", st, 12.0 * n * nrhs);
                    if (orow) op_cast_f32_rows(h->r0.get(), h->r0_32.get(), orow, n, nrhs, st);
                    else op_cast_f32(h->r0.get(), h->r0_32.get(), n * nrhs, st);
                }
                // the split-ordered correction may come back in two pieces
                const float *e_hi = vcycle<float>(h, 0, h->r0_32.get(), h->e32.get(), true,
                                                  nullptr, nrhs, st, orow != nullptr);
                {
                    ProfScope ps("cast", st, 20.0 * n * nrhs);
                    if (orow) op_axpy_f32_rows(x, h->e32.get(), orow, n, nrhs, st, e_hi, L0.nf);
                    else op_axpy_f32(x, h->e32.get(), n * nrhs, st);
                }
                residual_and_norms(st);
            });
        }
        read_norms(h->norms.get(), nrhs, s, rn);
        ++it;
    }
    if (vec_split) op_permute_rows(n, nrhs, L0.perm.get(), x, xu, false, s);
    LAIR_HIP(hipStreamSynchronize(s));
    if (info) {
        info->iters = it;
        info->relres = relmax;
        double rho = 0.0;
        if (it > 0 && !r_first.empty()) {
            for (int32_t q = 0; q < nrhs; ++q)
                if (r_first[q] > 0) rho = std::max(rho, std::pow(rn[q] / r_first[q], 1.0 / it));
        }
        info->rho = rho;
        info_common(h, info);
        set_history(info, hist);
        info->solve_ms = ms_since(t0);
    }
    return relmax <= rtol ? LAIR_OK : LAIR_ENOCONV;
}

// Flexible GMRES(m), right preconditioned (Saad 1993), with one V-cycle from
// zero as the preconditioner: the outer solver of the paper's results
// (Sec. 4).  Each right-hand side has its own Krylov space, Hessenberg
// matrix and Givens rotations (host), in shared device bases V (m + 1
// vectors) and Z (m vectors) of n x nrhs doubles in the natural ordering.
// Arnoldi: classical Gram-Schmidt applied twice.  A right-hand side whose
// residual estimate reaches rtol ||b|| is frozen (its next basis vectors are
// zero) and updated with its own number of steps; a cycle of m steps ends
// with the true residual, which decides whether to restart.
lair_status solve_fgmres_impl(lair_hierarchy *h, const double *b, double *x,
                              int32_t nrhs, double rtol, int32_t maxit, int32_t m,
                              lair_info *info, hipStream_t s) {
    auto t0 = Clock::now();
    check_solve_args(h, b, x, rtol, maxit);
    check_nrhs(h, nrhs);
    if (h->batch) fail(LAIR_EUNSUPPORTED, "FGMRES is for a single system");
    if (m < 1 || m > 64) fail(LAIR_EINVAL, "restart must be in [1, 64] (got %d)", m);
    ensure_vectors(h, nrhs, s);
    ensure_tail(h, nrhs, h->opt.precision == LAIR_MIXED, false, s);
    Level &L0 = *h->L[0];
    const int64_t n = L0.n;
    const int32_t R = nrhs;
    const int64_t nv = n * R;
    const bool mixed = h->opt.precision == LAIR_MIXED;
    const bool split = L0.split;
    const double *bb = b;
    if (scaled(h->opt)) {
        op_block_apply(n / h->opt.block_size, h->opt.block_size, h->dinv.get(), b,
                       h->bscaled.get(), nrhs, s);
        bb = h->bscaled.get();
    }
    CsrView<double> A0 = view<double>(L0.A, L0.team_A);
    DevArr<double> V, Z, w, coef, dots, partial;
    V.alloc((size_t)(m + 1) * nv, s);
    Z.alloc((size_t)m * nv, s);
    w.alloc((size_t)nv, s);
    coef.alloc((size_t)(m + 1) * R, s);
    // dots: both Gram-Schmidt passes' coefficients, then |w|^2
    const size_t HOFF = (size_t)(m + 1) * R;
    dots.alloc(2 * HOFF + R, s);
    partial.alloc((size_t)kry_dot_blocks(nv) * (m + 1) * R, s);
    double *Vp = V.get(), *Zp = Z.get();
    auto Vk = [&](int k) { return Vp + (int64_t)k * nv; };
    auto Zk = [&](int k) { return Zp + (int64_t)k * nv; };
    // z = B v: one V-cycle from zero, in the cycle's ordering and precision
    auto precond = [&](const double *v, double *z) {
        if (mixed) {
            if (split) op_cast_f32_rows(v, h->r0_32.get(), L0.iperm.get(), n, R, s);
            else op_cast_f32(v, h->r0_32.get(), nv, s);
            vcycle<float>(h, 0, h->r0_32.get(), h->e32.get(), true, nullptr, R, s);
            op_fill<double>(z, 0.0, nv, s);
            if (split) op_axpy_f32_rows(z, h->e32.get(), L0.iperm.get(), n, R, s);
            else op_axpy_f32(z, h->e32.get(), nv, s);
        } else if (split) {
            op_permute_rows(n, R, L0.perm.get(), v, h->bsplit.get(), true, s);
            vcycle<double>(h, 0, h->bsplit.get(), h->xsplit.get(), true, nullptr, R, s);
            op_permute_rows(n, R, L0.perm.get(), h->xsplit.get(), z, false, s);
        } else {
            vcycle<double>(h, 0, v, z, true, nullptr, R, s);
        }
    };
    auto upload = [&](double *dev, const std::vector<double> &hv) {
        double *st = (double *)pinned_upload(sizeof(double) * hv.size());
        memcpy(st, hv.data(), sizeof(double) * hv.size());
        LAIR_HIP(hipMemcpyAsync(dev, st, sizeof(double) * hv.size(), hipMemcpyHostToDevice, s));
        LAIR_HIP(hipStreamSynchronize(s));     // the staging area is reused
    };
    // r = b - A x into V_0 and its norms
    auto true_residual = [&](std::vector<double> &beta) {
        op_residual<double>(A0, bb, x, Vk(0), R, s);
        op_mdot(n, R, Vk(0), nv, 1, Vk(0), partial.get(), dots.get(), s);
        read_norms(dots.get(), R, s, beta);
    };
    std::vector<double> nb, beta, r_first;
    norms_host(h, bb, R, s, nb);
    std::vector<double> tol((size_t)R);
    for (int32_t q = 0; q < R; ++q) tol[q] = rtol * nb[q];
    true_residual(beta);
    r_first = beta;
    std::vector<int32_t> its((size_t)R, 0);
    const size_t H1 = (size_t)m + 1;
    std::vector<double> Hh(H1 * m * R), cs((size_t)m * R), sn((size_t)m * R), g(H1 * R);
    std::vector<double> hc(2 * HOFF + R), sc((size_t)R), cf((size_t)(m + 1) * R);
    std::vector<int32_t> kq((size_t)R);
    std::vector<char> act((size_t)R);
    int32_t it = 0;
    for (;;) {
        bool any = false;
        for (int32_t q = 0; q < R; ++q) {
            act[q] = !(beta[q] <= tol[q]);
            any = any || act[q];
        }
        if (!any || it >= maxit) break;
        // V_0 = r / beta for the right-hand sides still iterated
        for (int32_t q = 0; q < R; ++q) {
            sc[q] = act[q] ? 1.0 / beta[q] : 0.0;
            kq[q] = 0;
            g[q] = act[q] ? beta[q] : 0.0;
            for (size_t i = 1; i < H1; ++i) g[i * R + q] = 0.0;
        }
        op_scale_rhs(n, R, Vk(0), sc.data(), Vk(0), s);
        for (int j = 0; j < m; ++j) {
            precond(Vk(j), Zk(j));
            op_spmv<double>(A0, Zk(j), w.get(), R, false, s);
            // Gram-Schmidt twice: c = V^T w, w -= V c; h = c1 + c2
            double *c1 = dots.get(), *c2 = c1 + HOFF;
            op_mdot(n, R, Vp, nv, j + 1, w.get(), partial.get(), c1, s);
            op_gram_schmidt(n, R, Vp, nv, j + 1, c1, w.get(), true, partial.get(), c2, s);
            op_gram_schmidt(n, R, Vp, nv, j + 1, c2, w.get(), false, partial.get(), c2 + HOFF, s);
            {
                Readback rb(s);
                rb.add(hc.data(), dots.get(), sizeof(double) * (j + 1) * R);
                rb.add(hc.data() + HOFF, dots.get() + HOFF, sizeof(double) * (j + 1) * R);
                rb.add(hc.data() + 2 * HOFF, dots.get() + 2 * HOFF, sizeof(double) * R);
                rb.run();
            }
            for (int i = 0; i <= j; ++i)
                for (int32_t q = 0; q < R; ++q)
                    Hh[((size_t)i * m + j) * R + q] =
                        hc[(size_t)i * R + q] + hc[HOFF + (size_t)i * R + q];
            std::vector<double> hn((size_t)R);
            for (int32_t q = 0; q < R; ++q) hn[q] = std::sqrt(hc[2 * HOFF + q]);
            ++it;
            bool still = false;
            for (int32_t q = 0; q < R; ++q) {
                sc[q] = 0.0;
                if (!act[q]) continue;
                auto H = [&](size_t i, size_t jj) -> double & { return Hh[(i * m + jj) * R + q]; };
                H(j + 1, j) = hn[q];
                for (int i = 0; i < j; ++i) {
                    const double c = cs[(size_t)i * R + q], sg = sn[(size_t)i * R + q];
                    const double t = c * H(i, j) + sg * H(i + 1, j);
                    H(i + 1, j) = -sg * H(i, j) + c * H(i + 1, j);
                    H(i, j) = t;
                }
                const double d = std::hypot(H(j, j), H(j + 1, j));
                double c = 1.0, sg = 0.0;
                if (d > 0) { c = H(j, j) / d; sg = H(j + 1, j) / d; }
                cs[(size_t)j * R + q] = c;
                sn[(size_t)j * R + q] = sg;
                H(j, j) = d;
                H(j + 1, j) = 0.0;
                g[(size_t)(j + 1) * R + q] = -sg * g[(size_t)j * R + q];
                g[(size_t)j * R + q] = c * g[(size_t)j * R + q];
                kq[q] = j + 1;
                its[q] += 1;
                if (std::fabs(g[(size_t)(j + 1) * R + q]) <= tol[q]) {
                    act[q] = 0;          // frozen: its next basis vectors are zero
                } else {
                    still = true;
                    sc[q] = hn[q] > 0 ? 1.0 / hn[q] : 0.0;
                }
            }
            if (!still || it >= maxit || j + 1 == m) break;
            op_scale_rhs(n, R, w.get(), sc.data(), Vk(j + 1), s);
        }
        // x += Z y, y from the triangular systems (each right-hand side its
        // own number of steps; missing steps weigh zero)
        int kmax = 0;
        std::fill(cf.begin(), cf.end(), 0.0);
        for (int32_t q = 0; q < R; ++q) {
            const int k = kq[q];
            kmax = std::max(kmax, k);
            std::vector<double> y((size_t)k);
            for (int i = k - 1; i >= 0; --i) {
                double t = g[(size_t)i * R + q];
                for (int l = i + 1; l < k; ++l) t -= Hh[((size_t)i * m + l) * R + q] * y[l];
                y[i] = t / Hh[((size_t)i * m + i) * R + q];
            }
            for (int i = 0; i < k; ++i) cf[(size_t)i * R + q] = -y[i];
        }
        if (kmax > 0) {
            upload(coef.get(), cf);
            op_maxpy(n, R, Zp, nv, kmax, coef.get(), x, s);
        }
        true_residual(beta);
    }
    LAIR_HIP(hipStreamSynchronize(s));
    double relmax = 0.0;
    int32_t itmax = 0;
    for (int32_t q = 0; q < R; ++q) {
        relmax = std::max(relmax, nb[q] > 0 ? beta[q] / nb[q] : beta[q]);
        itmax = std::max(itmax, its[q]);
    }
    if (info) {
        info->iters = itmax;
        info->relres = relmax;
        double rho = 0.0;
        if (itmax > 0)
            for (int32_t q = 0; q < R; ++q)
                if (r_first[q] > 0 && its[q] > 0)
                    rho = std::max(rho, std::pow(beta[q] / r_first[q], 1.0 / its[q]));
        info->rho = rho;
        info_common(h, info);
        info->solve_ms = ms_since(t0);
    }
    return relmax <= rtol ? LAIR_OK : LAIR_ENOCONV;
}

// Longest run of a row list that one workgroup copies (whole runs, up to
// 102,400 rows, took 54 us a rebuild on 24 systems and 92 us on 512).
static const int32_t ACT_PIECE = 4096;

// The union's vectors that the systems' tails read and write.
static void set_batch_vectors(lair_hierarchy *h, bool mixed) {
    for (size_t l = 0; l < h->L.size(); ++l) {
        Level &Lv = *h->L[l];
        if (mixed) {
            auto &o = h->batch_tail->a32->lv[l];
            o.vb = l ? Lv.b32.get() : h->r0_32.get();
            o.vx = l ? Lv.x32.get() : h->e32.get();
        } else {
            auto &o = h->batch_tail->a64->lv[l];
            o.vb = l ? Lv.b.get() : h->r0.get();
            o.vx = l ? Lv.x.get() : h->e64.get();
        }
    }
}

// Batch of independent systems (one right-hand side each): the correction
// form x += B (b - A x) on the union, with the residual rows of converged
// systems zeroed so that their corrections vanish.  Each system stops at its
// own relative residual.
lair_status solve_batch_impl(lair_hierarchy *h, const double *b, double *x,
                             double rtol, int32_t maxit, int32_t *iters,
                             double *relres, lair_info *info, hipStream_t s) {
    auto t0 = Clock::now();
    check_solve_args(h, b, x, rtol, maxit);
    if (!h->batch) fail(LAIR_EINVAL, "the hierarchy was not built by lair_setup_batch");
    check_usable(h);
    ensure_vectors(h, 1, s);
    if (h->nsys == 1) ensure_tail(h, 1, h->opt.precision == LAIR_MIXED, false, s);
    Level &L0 = *h->L[0];
    const int32_t ns = h->nsys;
    const int64_t n = L0.n;
    bool mixed = h->opt.precision == LAIR_MIXED;
    // grow-only: captured iterations keep these addresses
    bool moved = false;
    if (h->seg_norm.get() == nullptr) { h->seg_norm.alloc((size_t)ns, s); moved = true; }
    if (h->active_dev.get() == nullptr) { h->active_dev.alloc((size_t)ns, s); moved = true; }
    if (!mixed && h->e64.get() == nullptr) { h->e64.alloc((size_t)n, s); moved = true; }
    // one system: the iteration stops when it converges, no lists needed
    const bool lists = ns > 1;
    const size_t cnt_bytes = (4 * sizeof(int32_t) * h->L.size() + 15) & ~(size_t)15;
    if (lists && L0.act_cnt == nullptr) {
        size_t maxseg = 4 * h->L.size() * (size_t)ns;
        for (auto &lp : h->L) maxseg += 4 * (size_t)lp->n / ACT_PIECE;
        h->act_upload.alloc(cnt_bytes + 8 * sizeof(void *) * h->L.size() +
                                sizeof(int32_t) * (4 * h->L.size() + 1 + 5 * maxseg), s);
        for (size_t l = 0; l < h->L.size(); ++l) {
            Level &Lv = *h->L[l];
            Lv.act_rows.alloc((size_t)std::max(Lv.n, 1), s);
            if (l + 1 < h->L.size()) {
                Lv.act_p.alloc((size_t)std::max(Lv.n, 1), s);
                Lv.act_f.alloc((size_t)std::max(Lv.nf, 1), s);
                Lv.act_c.alloc((size_t)std::max(Lv.nrc >= 0 ? Lv.nrc : Lv.nc, 1), s);
            }
        }
        // (what says that all of them are there, after an allocation failed too)
        for (size_t l = 0; l < h->L.size(); ++l)
            h->L[l]->act_cnt = reinterpret_cast<int32_t *>(h->act_upload.get()) + 4 * l;
        moved = true;
    }
    if (h->ss_nblk == 0) {
        // per-system norms: blocks of at most seg_sum_chunk() rows
        const int64_t ch = seg_sum_chunk();
        std::vector<int32_t> bsys;
        std::vector<int64_t> blo, bstart{0};
        for (int32_t q = 0; q < ns; ++q) {
            for (int64_t lo = L0.seg[q]; lo < L0.seg[q + 1]; lo += ch) {
                bsys.push_back(q);
                blo.push_back(lo);
            }
            bstart.push_back((int64_t)bsys.size());
        }
        h->ss_sys.alloc(bsys.size(), s);
        h->ss_lo.alloc(blo.size(), s);
        h->ss_start.alloc(bstart.size(), s);
        h->ss_part.alloc(bsys.size(), s);
        LAIR_HIP(hipMemcpyAsync(h->ss_sys.get(), bsys.data(), sizeof(int32_t) * bsys.size(),
                                hipMemcpyHostToDevice, s));
        LAIR_HIP(hipMemcpyAsync(h->ss_lo.get(), blo.data(), sizeof(int64_t) * blo.size(),
                                hipMemcpyHostToDevice, s));
        LAIR_HIP(hipMemcpyAsync(h->ss_start.get(), bstart.data(),
                                sizeof(int64_t) * bstart.size(), hipMemcpyHostToDevice, s));
        LAIR_HIP(hipStreamSynchronize(s));     // pageable sources
        h->ss_nblk = (int32_t)bsys.size();
        moved = true;
    }
    if (moved) h->drop_graphs();
    const size_t nlev = h->L.size();
    auto seg_norms = [&](const double *r, const uint8_t *act, hipStream_t st) {
        ProfScope ps("norm", st, 8.0 * n, 2.0 * n);
        launch_seg_sumsq_blocks(ns, h->ss_nblk, h->ss_sys.get(), h->ss_lo.get(),
                                h->ss_start.get(), L0.seg_dev.get(), act, r,
                                h->ss_part.get(), h->seg_norm.get(), st);
    };
    // rows of the systems still iterated, on every level.  A system's rows,
    // F rows and relaxed C rows are contiguous runs of the level's row range,
    // F list and relaxed-C list; a kernel lays out the runs of the active
    // systems and another copies them (no atomics, fixed order).
    std::vector<std::array<std::vector<int32_t>, 3>> runs(nlev);   // per list: prefix over systems
    for (size_t l = 0; lists && l < nlev; ++l) {
        Level &Lv = *h->L[l];
        for (int t = 0; t < 3; ++t) runs[l][t].assign((size_t)ns + 1, 0);
        const bool last = l + 1 == nlev;
        for (int32_t q = 0; q < ns; ++q) {
            const int32_t nq = (int32_t)(Lv.seg[q + 1] - Lv.seg[q]);
            int32_t cq = 0, rq = 0;
            if (!last) {
                cq = (int32_t)(Lv.next_seg[q + 1] - Lv.next_seg[q]);
                rq = Lv.stopped[q] ? 0 : cq;     // stopped systems' C rows are not relaxed
            }
            runs[l][0][q + 1] = runs[l][0][q] + nq;
            runs[l][1][q + 1] = runs[l][1][q] + (last ? 0 : nq - cq);
            runs[l][2][q + 1] = runs[l][2][q] + rq;
        }
    }
    // the systems' tails, one workgroup each
    if (lists && !h->batch_tail) {
        h->batch_tail = unless_no_memory([&] {
            return mixed ? make_batch_tail<float>(h, runs, s)
                         : make_batch_tail<double>(h, runs, s);
        });
        if (!h->batch_tail) {
            h->batch_tail.reset(new Tail());      // none: past every level
            h->batch_tail->start = nlev;
            h->batch_tail->top.assign((size_t)ns, (int32_t)nlev);
        }
        h->drop_graphs();
    }
    if (lists) repack(*h->batch_tail, s);
    const std::vector<int32_t> no_top;
    const std::vector<int32_t> &top = lists ? h->batch_tail->top : no_top;
    // the runs of every list, laid end to end, as the device holds them:
    // where each list begins, then each run's system, list, start and length
    // (long runs in pieces).  When systems stop the host uploads their flags
    // alone.  (Laid out by the host after every stop: 512 systems, 32 stops, 92
    // us each before the copy; on the device 7 us.)
    const int32_t nlists = 4 * (int32_t)nlev;
    int32_t nruns = 0;
    const int32_t **d_src = nullptr;
    int32_t **d_dst = nullptr;
    int32_t *run_ptr = nullptr, *run_sys = nullptr, *run_list = nullptr, *run_start = nullptr,
            *run_len = nullptr, *run_dst = nullptr;
    if (lists) {
        std::vector<int32_t> ptr{0}, sys, list, start, len;
        for (size_t l = 0; l < nlev; ++l)
            for (int t = 0; t < 4; ++t) {
                const int k = t == 3 ? 0 : t;
                for (int32_t q = 0; q < ns && (t == 0 || l + 1 < nlev); ++q) {
                    // a system's tail takes its right-hand side at level
                    // top[q] and does the rest from there
                    if ((size_t)top[q] + (t == 0) <= l) continue;
                    const int32_t m = runs[l][k][q + 1] - runs[l][k][q];
                    const int32_t s0 = k == 0 ? (int32_t)h->L[l]->seg[q] : runs[l][k][q];
                    for (int32_t o = 0; o < m; o += ACT_PIECE) {
                        sys.push_back(q);
                        list.push_back((int32_t)(4 * l + t));
                        start.push_back(s0 + o);
                        len.push_back(std::min(ACT_PIECE, m - o));
                    }
                }
                ptr.push_back((int32_t)sys.size());
            }
        nruns = (int32_t)sys.size();
        d_src = reinterpret_cast<const int32_t **>(h->act_upload.get() + cnt_bytes);
        d_dst = const_cast<int32_t **>(d_src) + nlists;
        run_ptr = reinterpret_cast<int32_t *>(d_dst + nlists);
        run_sys = run_ptr + nlists + 1;
        run_list = run_sys + nruns;
        run_start = run_list + nruns;
        run_len = run_start + nruns;
        run_dst = run_len + nruns;
        // where the lists come from and go to, and the runs, in one copy from
        // pinned memory (free again when the systems' flags are uploaded:
        // readbacks come between).  Three pageable copies and a wait for them
        // took 25 us of the 175 that a solve of 400 grids of 6 x 6 took.
        const size_t bytes = 2 * sizeof(void *) * nlists + sizeof(int32_t) * (nlists + 1 + 4 * (size_t)nruns);
        char *st = (char *)pinned_upload(bytes), *at = st;
        auto put = [&at](const void *from, size_t n) {
            memcpy(at, from, n);
            at += n;
        };
        std::vector<const int32_t *> from((size_t)nlists, nullptr), to((size_t)nlists, nullptr);
        for (size_t l = 0; l < nlev; ++l) {
            Level &Lv = *h->L[l];
            to[4 * l] = Lv.act_rows.get();
            if (l + 1 < nlev) {
                from[4 * l + 1] = Lv.flist.get();
                to[4 * l + 1] = Lv.act_f.get();
                from[4 * l + 2] = Lv.nrc >= 0 ? Lv.rclist.get() : Lv.clist.get();
                to[4 * l + 2] = Lv.act_c.get();
                to[4 * l + 3] = Lv.act_p.get();
            }
        }
        put(from.data(), sizeof(void *) * from.size());
        put(to.data(), sizeof(void *) * to.size());
        for (const auto *v : {&ptr, &sys, &list, &start, &len})
            put(v->data(), sizeof(int32_t) * v->size());
        LAIR_HIP(hipMemcpyAsync(h->act_upload.get() + cnt_bytes, st, bytes,
                                hipMemcpyHostToDevice, s));
    }
    auto rebuild_lists = [&]() {
        launch_active_lists(nlists, nruns, run_ptr, run_sys, run_list, run_start, run_len,
                            run_dst, h->active_dev.get(), L0.act_cnt, d_src, d_dst, s);
    };
    struct ActGuard {
        lair_hierarchy *h;
        ~ActGuard() { h->use_act = false; }
    } act_guard{h};
    const double *bb = b;
    if (scaled(h->opt)) {
        op_block_apply(n / h->opt.block_size, h->opt.block_size, h->dinv.get(), b,
                       h->bscaled.get(), 1, s);
        bb = h->bscaled.get();
    }
    std::vector<double> nb, rn, rfirst;
    seg_norms(bb, nullptr, s);
    read_norms(h->seg_norm.get(), ns, s, nb);
    CsrView<double> A0 = view<double>(L0.A, L0.team_A);
    auto residual_and_norms = [&](hipStream_t st) {
        {
            ProfScope ps("residual", st, ab_rowdot(L0.A, 8, 1, 2), 2.0 * L0.A.nnz);
            op_residual<double>(A0, bb, x, h->r0.get(), 1, st);
        }
        seg_norms(h->r0.get(), nullptr, st);
    };
    residual_and_norms(s);
    // later residuals are written with their float copy
    if (mixed && lists) op_cast_f32(h->r0.get(), h->r0_32.get(), n, s);
    read_norms(h->seg_norm.get(), ns, s, rn);
    rfirst = rn;
    h->active.assign((size_t)ns, 1);
    std::vector<int32_t> its((size_t)ns, 0);
    std::vector<double> rel((size_t)ns, 0.0);
    bool upload = true;
    int32_t it = 0;
    std::vector<double> hist;
    for (;;) {
        int32_t nact = 0;
        for (int32_t q = 0; q < ns; ++q) {
            if (!h->active[q]) continue;
            rel[q] = nb[q] > 0 ? rn[q] / nb[q] : rn[q];
            its[q] = it;
            if (rel[q] <= rtol) {
                h->active[q] = 0;
                upload = true;
            } else {
                ++nact;
            }
        }
        hist.push_back(*std::max_element(rel.begin(), rel.end()));
        if (nact == 0 || it >= maxit) break;
        if (upload) {
            // (the pinned area is free: a readback has followed its last use)
            void *st = pinned_upload((size_t)ns);
            memcpy(st, h->active.data(), (size_t)ns);
            LAIR_HIP(hipMemcpyAsync(h->active_dev.get(), st, (size_t)ns,
                                    hipMemcpyHostToDevice, s));
            if (lists) rebuild_lists();
            upload = false;
        }
        // the cycle touches only the rows of systems still iterated; the
        // others keep their x (their corrections would be zero)
        h->use_act = lists;
        if (lists && h->batch_tail->start < nlev) set_batch_vectors(h, mixed);
        run_iteration(h, mixed ? IT_BATCH_MIXED : IT_BATCH_FP64, 1, bb, x, s,
                      [&](hipStream_t st) {
            if (mixed) {
                if (!lists) {
                    ProfScope ps("cast", st, 12.0 * n);
                    op_cast_f32(h->r0.get(), h->r0_32.get(), n, st);
                }
                vcycle<float>(h, 0, h->r0_32.get(), h->e32.get(), true, nullptr, 1, st);
                ProfScope ps("cast", st, 20.0 * n);
                if (lists)
                    op_update_list<float>(L0.act_rows.get(), L0.act_cnt, (int32_t)n, x,
                                          h->e32.get(), st);
                else
                    op_axpy_f32(x, h->e32.get(), n, st);
            } else {
                vcycle<double>(h, 0, h->r0.get(), h->e64.get(), true, nullptr, 1, st);
                if (lists) {
                    op_update_list<double>(L0.act_rows.get(), L0.act_cnt, (int32_t)n, x,
                                           h->e64.get(), st);
                } else {
                    LAIR_LAUNCH(k_add, dim3(blocks_for(n, 256)), dim3(256), 0, st, x,
                                h->e64.get(), n);
                    LAIR_LAUNCH_CHECK();
                }
            }
            {
                ProfScope ps("residual", st, ab_rowdot(L0.A, 8, 1, 2), 2.0 * L0.A.nnz);
                if (lists)
                    op_residual_list(A0, L0.act_rows.get(), L0.act_cnt, (int32_t)n, x, bb,
                                     h->r0.get(), mixed ? h->r0_32.get() : nullptr, st);
                else
                    op_residual<double>(A0, bb, x, h->r0.get(), 1, st);
            }
            seg_norms(h->r0.get(), h->active_dev.get(), st);
        });
        h->use_act = false;
        read_norms(h->seg_norm.get(), ns, s, rn);
        ++it;
    }
    LAIR_HIP(hipStreamSynchronize(s));
    double relmax = 0.0;
    int32_t itmax = 0;
    bool conv = true;
    for (int32_t q = 0; q < ns; ++q) {
        if (iters) iters[q] = its[q];
        if (relres) relres[q] = rel[q];
        relmax = std::max(relmax, rel[q]);
        itmax = std::max(itmax, its[q]);
        conv = conv && rel[q] <= rtol;
    }
    if (info) {
        info->iters = itmax;
        info->relres = relmax;
        double rho = 0.0;
        for (int32_t q = 0; q < ns; ++q)
            if (its[q] > 0 && rfirst[q] > 0)
                rho = std::max(rho, std::pow(rel[q] * nb[q] / rfirst[q], 1.0 / its[q]));
        info->rho = rho;
        info_common(h, info);
        set_history(info, hist);
        info->solve_ms = ms_since(t0);
    }
    return conv ? LAIR_OK : LAIR_ENOCONV;
}

// ---------------------------------------------------------------------------
// One cycle from a given iterate (lair_cycle) and its transpose
// ---------------------------------------------------------------------------
void cycle_impl(lair_hierarchy *h, const double *b, double *x, int32_t nrhs, hipStream_t s) {
    if (!h || !b || !x) fail(LAIR_EINVAL, "NULL argument");
    check_nrhs(h, nrhs);
    ensure_vectors(h, nrhs, s);
    ensure_tail(h, nrhs, h->opt.precision == LAIR_MIXED, false, s);
    cycle_body(h, b, x, nrhs, s);
}

void cycle_body(lair_hierarchy *h, const double *b, double *x, int32_t nrhs, hipStream_t s) {
    const double *bb = b;
    int64_t n = h->L[0]->n;
    if (scaled(h->opt)) {
        op_block_apply(n / h->opt.block_size, h->opt.block_size, h->dinv.get(), b,
                       h->bscaled.get(), nrhs, s);
        bb = h->bscaled.get();
    }
    Level &L0 = *h->L[0];
    if (h->opt.precision == LAIR_MIXED) {
        op_residual<double>(view<double>(L0.A, L0.team_A), bb, x, h->r0.get(), nrhs, s);
        if (L0.split) op_cast_f32_rows(h->r0.get(), h->r0_32.get(), L0.iperm.get(), n,
                                       nrhs, s);
        else op_cast_f32(h->r0.get(), h->r0_32.get(), n * nrhs, s);
        vcycle<float>(h, 0, h->r0_32.get(), h->e32.get(), true, nullptr, nrhs, s);
        if (L0.split) op_axpy_f32_rows(x, h->e32.get(), L0.iperm.get(), n, nrhs, s);
        else op_axpy_f32(x, h->e32.get(), n * nrhs, s);
    } else if (L0.split) {
        op_permute_rows(n, nrhs, L0.perm.get(), bb, h->bsplit.get(), true, s);
        op_permute_rows(n, nrhs, L0.perm.get(), x, h->xsplit.get(), true, s);
        vcycle<double>(h, 0, h->bsplit.get(), h->xsplit.get(), false, nullptr, nrhs, s);
        op_permute_rows(n, nrhs, L0.perm.get(), h->xsplit.get(), x, false, s);
    } else {
        vcycle<double>(h, 0, bb, x, false, nullptr, nrhs, s);
    }
}

void cycle_transpose_impl(lair_hierarchy *h, const double *g, double *lam, int32_t nrhs,
                          hipStream_t s) {
    if (!h || !g || !lam) fail(LAIR_EINVAL, "NULL argument");
    check_nrhs(h, nrhs);
    if (nodal(h->opt)) fail(LAIR_EUNSUPPORTED, "transposed cycle on a nodal hierarchy");
    ensure_vectors(h, nrhs, s);
    ensure_transposes(h, s);
    ensure_tail(h, nrhs, false, true, s);
    // lam <- lam + B^T (g - A^T lam)
    Level &L0 = *h->L[0];
    int64_t n = L0.n;
    op_residual<double>(view<double>(L0.At, L0.team_At), g, lam, h->r0.get(), nrhs, s);
    vcycle_t(h, 0, h->r0.get(), L0.b.get(), nrhs, s);
    LAIR_LAUNCH(k_add, dim3(blocks_for(n * nrhs, 256)), dim3(256), 0, s,
                       lam, L0.b.get(), n * nrhs);
    LAIR_LAUNCH_CHECK();
}

}  // namespace lair
