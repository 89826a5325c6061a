// tail.hpp -- the bottom of a V-cycle in one workgroup (k_tail.hip): its
// packed operators, the tables its kernels read, and their launchers.
#pragma once

#include <hip/hip_runtime.h>

#include <cstddef>
#include <cstdint>
#include <vector>

namespace lair {

constexpr int TAIL_MAX_LEVELS = 20;     // the table is a kernel argument (4 KB)

// The row sets of a level that the tail sums: restriction rows (of the next
// level), interpolation rows, F rows and C rows of the sweeps, and every row
// (residual).
enum { TAIL_R = 0, TAIL_P = 1, TAIL_F = 2, TAIL_C = 3, TAIL_A = 4, TAIL_SETS = 5 };

// One row set, packed for the lanes that sum it.  A chunk is what one wave
// sums at once: 64 >> lg rows, 2^lg lanes each.  A lane's share of its row
// is stored in groups of U entries, U = 1 or 4; the lanes of a chunk lie side
// by side in each group, columns (16-bit, local to the system) apart from
// values.  Every address follows from the chunk's number, so a wave loads a
// chunk without reading a row pointer first.  In the blob, for nchunk chunks
// of at most smax groups: groups used (uint16 each), and for F and C rows the
// row and its diagonal entry per lane, then columns, then values.
struct TailSet {
    uint32_t o_used, o_row, o_diag, o_col, o_val;   // places of the parts in the blob
    uint16_t smax;
    uint8_t lg, u4;                     // u4: groups of four
};

template <class VT>
struct TailLevel {
    TailSet set[TAIL_SETS];
    const double *dinv;                 // nodal: inverse diagonal blocks
    // batch: row offsets of the systems here, of their runs in the F and C
    // lists, their first chunks per set ([set][nsys + 1]), and the union's
    // vectors of this level
    const int64_t *seg;
    const int32_t *frun, *crun, *chunk0;
    const VT *vb;
    VT *vx;
    int32_t n, nf, nc;                  // rows, F rows, C rows (of the union)
};

template <class VT>
struct TailArgs {
    int32_t nlv;                        // levels, the coarsest included
    int32_t nrhs;                       // right-hand sides (single system)
    int32_t knode;                      // nodal block size, or 0
    int32_t lds_bytes;                  // work vectors
    VT omega;
    const char *blob;                   // the packed sets
    const double *kinv;                 // coarsest inverse (single system)
    // batch (order != nullptr): the systems by decreasing size, the level each
    // system's tail starts at, its number of levels, its coarsest inverse
    const int32_t *order, *top, *slev;
    const int64_t *doff;
    const double *binv;
    const uint8_t *active;
    int32_t nsys;
    TailLevel<VT> lv[TAIL_MAX_LEVELS];
};

// Source of one packed set: CSR rows (listed, or 0 .. n - 1), taken by teams
// of 2^lg lanes with 2^ll consecutive entries a step.
template <class VT>
struct TailSource {
    const int32_t *rp, *cj;
    const VT *v;
    const int32_t *rows;                // or nullptr
    // batch: row (list position) offsets and column offsets of the systems
    const int32_t *run;                 // listed rows
    const int64_t *rseg, *cseg;
    const int32_t *chunk0;
    int32_t n, ncol, nchunk, nsys;
    uint8_t lg, ll, diag;
    TailSet dst;
};

template <class VT>
struct TailSources {
    char *blob;
    TailSource<VT> src[TAIL_SETS];
};

// What the tail starts from: a zero iterate and the right-hand side b (x
// assigned), an iterate x with its residual r given, or an iterate x alone.
enum { TAIL_ZERO = 0, TAIL_RESID = 1, TAIL_ITERATE = 2 };

// chunks of n rows taken by 2^lg lanes each
inline int32_t tail_chunks(int32_t n, int lg) {
    return (int32_t)((((int64_t)n << lg) + 63) / 64);
}
// groups that a row of up to max_row entries takes per lane
int32_t tail_groups(int32_t max_row, int lg, int ll, bool u4);
// place the parts of a set (smax and u4 given) of w-byte values from `at` on;
// returns where the next set may begin
size_t tail_layout(TailSet &t, size_t at, int32_t nchunk, bool rows, size_t w);
// pack every set of the levels (sets with nchunk = 0 are left out)
template <class VT>
void launch_tail_pack(const std::vector<TailSources<VT>> &levels, hipStream_t s);
template <class VT>
void launch_tail(const TailArgs<VT> &a, int mode, const VT *b, VT *x, const VT *r,
                 hipStream_t s);
// lam = B^T g from zero (the transposed operators in the table: A^T in the
// sweeps and the residual, P^T as restriction, R^T as interpolation)
void launch_tail_t(const TailArgs<double> &a, const double *g, double *lam, hipStream_t s);
// dynamic LDS one workgroup may ask for
size_t tail_lds_limit();
// longest row of each of the m CSR matrices (rp[k], nrows[k]); waits for s
void max_rows(int m, const int32_t *const *rp, const int32_t *nrows, int32_t *out,
              hipStream_t s);

}  // namespace lair
