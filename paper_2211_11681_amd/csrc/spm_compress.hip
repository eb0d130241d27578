// Samplet compression of a Matern kernel matrix on the device (Section 3.3):
// vals = P_S(T K T^T), evaluated exactly with O(N^2) kernel evaluations.
//
// T is never formed.  Its action is the two-scale transform of Section 3.2 applied
// in place: every cluster maps the values at its input slots (its points for a
// leaf, the scaling slots of its two sons otherwise) by Q^T, writing output k to
// input slot k; the first outputs are the scaling coefficients handed up, the rest
// are samplet coefficients.
//
// The tree is cut into stages.  A subtree of stage 1 is a largest one with at most
// kBlk points; of stage j + 1, a largest one whose stage-j subtrees hand up at most kSub
// scaling coefficients.  All clusters of a subtree that no earlier stage covers are
// transformed in one pass with the subtree's inputs in LDS, leaves first, every cluster's
// product with Q on the matrix cores.
//
// K is processed in panels of rows: the rows of one subtree (points p0 .. p0+rows).
//   1. W = the panel's kernel values with stage 1 of the column transform applied: a
//      workgroup evaluates the block of one stage-1 subtree's rows and another's columns
//      in LDS, transforms its columns there and writes it once
//   2. the later stages of the column transform on the scaling columns of W, then stage 1
//      of the row transform (where the columns have one stage only, it is part of step 1)
//   3. the panel's upper clusters combine the scaling rows of W, leaves first
//   4. extract:         samplet rows of the subtree's clusters -> tiles on S
//   5. the subtree root's scaling rows move to a buffer U
// After all panels the clusters above the panel level combine rows of U the same
// way (steps 3 and 4 on U).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <mutex>
#include <new>
#include <set>
#include <vector>

#include "spm_internal.h"

using spm::fail;

namespace {

constexpr int kMaxIn = 64;    // largest number of inputs of one cluster transform
constexpr int kBlk = 64;      // points of a stage-1 subtree
constexpr int kSub = 256;     // inputs of a subtree of a later stage
constexpr int kBlkX = kBlk + 4;   // row strides of the LDS tiles: 16 rows of a column then
constexpr int kPad = 4;           // fall into different banks
constexpr int kStageT = 512;  // threads of the later stages
constexpr int kRowC = 32;     // columns per workgroup of the panels' upper row transform
constexpr int kRowR = 256;    // rows it can hold

struct KParams {
    double c[4];     // polynomial P(s) coefficients, degree p
    int p;
    double sfac;     // s = sfac * r, sfac = sqrt(2p+1) / ell
    double ell, scale;
    int deriv;
};

template <int P>
__device__ inline double kernel_value(double r, const KParams &kp)
{
    const double s = kp.sfac * r;
    double poly = 0.0, dpoly = 0.0;
#pragma unroll
    for (int k = P; k >= 0; --k) poly = fma(poly, s, kp.c[k]);
#pragma unroll
    for (int k = P; k >= 1; --k) dpoly = fma(dpoly, s, k * kp.c[k]);
    const double ex = exp(-s);
    if (!kp.deriv) return kp.scale * ex * poly;
    return kp.scale * (-s / kp.ell) * (dpoly - poly) * ex;
}

// ------------------------------------------------------------------ cluster transforms in LDS
// One cluster's transform: its matrix fragments (at foff), m inputs and outputs, and where
// the inputs are among its subtree's: input k is base0 + k below n0 and base1 + k - n0 from
// there on.  Two runs are enough: a leaf's inputs are its points; another cluster's are the
// scaling coefficients of its two sons, and those of a cluster are the first of its own
// inputs, which lie in its first run, unless the whole first son is handed up, whose run
// the second one then continues.
struct ClusterRec {
    int64_t foff;
    int32_t m, n0, base0, base1;
    __host__ __device__ int operator()(int k) const { return k < n0 ? base0 + k : base1 + (k - n0); }
};

// Device tables of the stages.  Subtree u has the inputs in_off[u] .. in_off[u + 1] (their
// slots in_pos) and the levels lv_off[u] .. lv_off[u + 1] - 1, deepest first, level l the
// clusters lv_start[l] .. lv_start[l + 1] of rec.
struct StageTab {
    const ClusterRec *rec;
    const int64_t *in_off, *lv_off, *lv_start, *in_pos;
    const double *f;                  // matrix fragments (frag_index)
};

typedef double dbl4 __attribute__((ext_vector_type(4)));

// The transform matrix M (row k: output k's coefficients over the inputs) is stored as the
// MFMA operands that its product takes, zero outside: element [16 kb + l % 16][4 t + l / 16]
// for lane l, step t and output block kb, so a step is one coalesced load and no vector
// instruction.  (Those exclude the MFMAs on a SIMD: with m x m matrices, bounds tests and
// index lists the transforms of a kernel block took 229 us per panel of N = 65536, against
// 60 us of MFMAs.)
__host__ __device__ inline int64_t frag_index(int m, int kb, int t) { return ((int64_t)kb * ((m + 3) >> 2) + t) * 64; }

// The fragments of cluster blockIdx.x, at foff: M = Q^T (Q column-major, so M[k][i] = q[k m + i]),
// or the inverse transform's Q.  Formed here, as on the host they took most of a tree's first
// transform (N = 60000: 15.6 ms, of which the first transform's own work is 0.03 ms).
__global__ void k_fragments(const int32_t *__restrict__ nin, const int64_t *__restrict__ qoff,
                            const int64_t *__restrict__ foff, const double *__restrict__ qmat, double *__restrict__ f,
                            bool inv)
{
    const int c = blockIdx.x, m = nin[c], nt = (m + 3) >> 2;
    const double *q = qmat + qoff[c];
    double *o = f + foff[c];
    for (int e = threadIdx.x; e < (m + 15) / 16 * nt * 64; e += blockDim.x) {
        const int l = e & 63, b = e >> 6, k = 16 * (b / nt) + l % 16, i = 4 * (b % nt) + l / 16;
        o[e] = k < m && i < m ? (inv ? q[i * m + k] : q[k * m + i]) : 0.0;
    }
}

// One cluster's transform of NB blocks of 16 rows (columns) of a tile of row stride X, in
// place, by one wave: all results (up to NT k steps of four inputs, as many outputs) are
// formed in registers before the first one is written.  COLS: the cluster's inputs are the tile columns
// loc(k), and rows r0 .. are transformed (out[r][k] = sum_i in[r][i] M[k][i]); else the
// tile rows loc(k), and columns r0 ...  lim: rows (columns) of the tile.  RUN: the inputs
// are one run.
template <int NT, int NB, bool COLS, bool RUN>
__device__ __forceinline__ void cluster_task(double *tile, int X, int r0, int lim, const double *__restrict__ F,
                                             const ClusterRec &loc, int lane)
{
    const int m = loc.m, nt = (m + 3) >> 2, lr = lane & 15, lk = lane >> 4;
    constexpr int KB = (NT + 3) / 4;
    constexpr bool AHEAD = NT <= 8;                    // all fragments loaded before the MFMAs
    double f[AHEAD ? NT : 1][KB];
    if constexpr (AHEAD) {
#pragma unroll
        for (int t = 0; t < NT; ++t)
#pragma unroll
            for (int kb = 0; kb < KB; ++kb)
                if (t < nt && 16 * kb < m) f[t][kb] = F[(uint32_t)(frag_index(m, kb, t) + lane)];
    }
    dbl4 acc[KB][NB];
#pragma unroll
    for (int kb = 0; kb < KB; ++kb)
#pragma unroll
        for (int b = 0; b < NB; ++b) acc[kb][b] = dbl4{0.0, 0.0, 0.0, 0.0};
    const int si = COLS ? 1 : X, sr = COLS ? X : 1;    // strides of an input, of a row or column
    const double *rp[NB], *run[NB];
#pragma unroll
    for (int b = 0; b < NB; ++b) {
        rp[b] = tile + min(r0 + 16 * b + lr, lim - 1) * sr;
        run[b] = rp[b] + (loc.base0 + lk) * si;
    }
    auto step = [&](int t, const double (&ft)[KB]) {
        // the last step's rows past m are zeros, as their coefficients are (0 x inf is none)
        const bool whole = RUN && 4 * t + 3 < m;
        const int li = whole ? 0 : loc(min(4 * t + lk, m - 1)) * si;
#pragma unroll
        for (int b = 0; b < NB; ++b) {
            double in = whole ? run[b][4 * t * si] : rp[b][li];
            if (4 * t + 3 >= m && 4 * t + lk >= m) in = 0.0;
#pragma unroll
            for (int kb = 0; kb < KB; ++kb)
                if (16 * kb < m)
                    acc[kb][b] = COLS ? __builtin_amdgcn_mfma_f64_16x16x4f64(in, ft[kb], acc[kb][b], 0, 0, 0)
                                      : __builtin_amdgcn_mfma_f64_16x16x4f64(ft[kb], in, acc[kb][b], 0, 0, 0);
        }
    };
    if constexpr (AHEAD) {
#pragma unroll
        for (int t = 0; t < NT; ++t)
            if (t < nt) step(t, f[t]);
    } else {
        for (int t = 0; t < nt; ++t) {
#pragma unroll
            for (int kb = 0; kb < KB; ++kb)
                if (16 * kb < m) f[0][kb] = F[(uint32_t)(frag_index(m, kb, t) + lane)];
            step(t, f[0]);
        }
    }
    // register r of a result: row 4r + lk, column lr (COLS: row of the tile, output k)
#pragma unroll
    for (int kb = 0; kb < KB; ++kb) {
        if (16 * kb >= m) continue;
        if constexpr (COLS) {
            const int k = 16 * kb + lr;
            double *const o = tile + (RUN ? loc.base0 + k : loc(min(k, m - 1))) + (r0 + lk) * X;
            if (k < m)
#pragma unroll
                for (int b = 0; b < NB; ++b)
#pragma unroll
                    for (int r = 0; r < 4; ++r)
                        if (r0 + 16 * NB <= lim || r0 + 16 * b + 4 * r + lk < lim) o[(16 * b + 4 * r) * X] = acc[kb][b][r];
        } else {
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int k = 16 * kb + 4 * r + lk;
                double *const o = tile + (RUN ? loc.base0 + k : loc(min(k, m - 1))) * X + r0 + lr;
                if (16 * kb + 16 <= m || k < m)
#pragma unroll
                    for (int b = 0; b < NB; ++b)
                        if (r0 + 16 * NB <= lim || r0 + 16 * b + lr < lim) o[16 * b] = acc[kb][b][r];
            }
        }
    }
}

// All clusters of subtree u on a tile in LDS, a level at a time; the waves take pairs
// (cluster, NB blocks of 16 of the lim rows or columns) in turn.  Starts and ends with the
// tile complete (barriers).  inv: the inverse transform, root first.
template <int NB, bool COLS>
__device__ __forceinline__ void subtree_transform(const StageTab &T, int64_t u, double *tile, int X, int lim, bool inv)
{
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int nw = blockDim.x >> 6, nb = (lim + 16 * NB - 1) / (16 * NB);
    const int64_t l0 = T.lv_off[u], l1 = T.lv_off[u + 1] - 1;
    for (int64_t l = 0; l < l1 - l0; ++l) {
        const int64_t lv = inv ? l1 - 1 - l : l0 + l;
        const int64_t a = T.lv_start[lv], cnt = T.lv_start[lv + 1] - a;
        __syncthreads();
        for (int w = wave; w < (int)cnt * nb; w += nw) {
            const ClusterRec loc = T.rec[a + w / nb];
            const int m = loc.m, r0 = (w % nb) * 16 * NB;
            const double *F = T.f + loc.foff;
            const bool run = loc.n0 >= m;
            if (m <= 16) {
                if (run) cluster_task<4, NB, COLS, true>(tile, X, r0, lim, F, loc, lane);
                else cluster_task<4, NB, COLS, false>(tile, X, r0, lim, F, loc, lane);
            } else if (m <= 32) {
                if (run) cluster_task<8, NB, COLS, true>(tile, X, r0, lim, F, loc, lane);
                else cluster_task<8, NB, COLS, false>(tile, X, r0, lim, F, loc, lane);
            } else                                     // one block at a time: more do not fit the registers
                for (int b = 0; b < NB; ++b)
                    if (r0 + 16 * b < lim)
                        cluster_task<kMaxIn / 4, 1, COLS, false>(tile, X, r0 + 16 * b, lim, F, loc, lane);
        }
    }
    __syncthreads();
}

// Kernel block of the rows of subtree sub0 + blockIdx.y and the columns of subtree
// blockIdx.x (both of stage 1), its columns transformed, to rows p0 .. of W; the rows as well
// (both) where the tree has no later column stage.  With one, the rows wait for it: a column
// stage after them would round row scaling coefficients, larger than the kernel values by
// the root of their points' number, which shows where fine rows meet coarse columns
// (million-point square: 1.4e-12 of the sampled entries' norm, 0.8e-12 in this order).
// Bound by the vector unit (distance, square root, exponential) and the matrix products,
// which exclude each other: about 7 and 8 ms of N = 65536 with both sides.
template <int P>
__global__ __launch_bounds__(256, 4) void k_eval_block(double *__restrict__ W, const double *__restrict__ pts, int d,
                                                       int64_t p0, int64_t n, int64_t sub0, KParams kp, StageTab T, bool both)
{
    __shared__ double tile[kBlk * kBlkX];
    const int64_t rs = sub0 + blockIdx.y, cs = blockIdx.x;
    const int64_t r0 = T.in_pos[T.in_off[rs]], c0 = T.in_pos[T.in_off[cs]];
    const int nr = (int)(T.in_off[rs + 1] - T.in_off[rs]), nc = (int)(T.in_off[cs + 1] - T.in_off[cs]);
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    {
        double y[3];
        const int64_t q = c0 + min(lane, nc - 1);
#pragma unroll
        for (int a = 0; a < 3; ++a) y[a] = a < d ? pts[q * d + a] : 0.0;
        for (int r = wave; r < nr; r += 4) {
            const double *x = pts + (r0 + r) * d;      // the wave's row: scalar loads
            double acc = 0.0;
#pragma unroll
            for (int a = 0; a < 3; ++a)
                if (a < d) {
                    const double df = x[a] - y[a];
                    acc = fma(df, df, acc);
                }
            if (lane < nc) tile[r * kBlkX + lane] = kernel_value<P>(sqrt(acc), kp);
        }
    }
    subtree_transform<2, true>(T, cs, tile, kBlkX, nr, false);
    if (both) subtree_transform<2, false>(T, rs, tile, kBlkX, nc, false);
    for (int r = wave; r < nr; r += 4)
        if (lane < nc) W[(r0 - p0 + r) * n + c0 + lane] = tile[r * kBlkX + lane];
}

// Row transform of stage 1 in place: the rows of subtree sub0 + blockIdx.y, 64 columns.
__global__ __launch_bounds__(256, 4) void k_rows_block(double *__restrict__ W, int64_t p0, int64_t n, int64_t sub0, StageTab T)
{
    __shared__ double tile[kBlk * kBlkX];
    const int64_t rs = sub0 + blockIdx.y, r0 = T.in_pos[T.in_off[rs]], c0 = (int64_t)blockIdx.x * kBlk;
    const int nr = (int)(T.in_off[rs + 1] - T.in_off[rs]), nc = (int)min<int64_t>(kBlk, n - c0);
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    double *const P = W + (r0 - p0) * n + c0;
#pragma unroll 8
    for (int r = wave; r < nr; r += 4)
        if (lane < nc) tile[r * kBlkX + lane] = P[r * n + lane];
    subtree_transform<2, false>(T, rs, tile, kBlkX, nc, false);
    for (int r = wave; r < nr; r += 4)
        if (lane < nc) P[r * n + lane] = tile[r * kBlkX + lane];
}

// Column transform of one later stage on 16 rows of W, in place: subtree sub0 + blockIdx.x.
__global__ __launch_bounds__(kStageT) void k_cols_stage(double *__restrict__ W, int64_t rows, int64_t n, int64_t sub0,
                                                    StageTab T)
{
    extern __shared__ double tile[];
    const int64_t u = sub0 + blockIdx.x, i0 = T.in_off[u], row0 = (int64_t)blockIdx.y * 16;
    const int ni = (int)(T.in_off[u + 1] - i0), X = ni + kPad, nr = (int)min<int64_t>(16, rows - row0);
    const int ti = threadIdx.x & 63, tr = threadIdx.x >> 6;   // lanes over the inputs, waves over the rows
#pragma unroll 4
    for (int i = ti; i < ni; i += 64) {
        const int64_t pos = T.in_pos[i0 + i];
        for (int r = tr; r < nr; r += kStageT / 64) tile[r * X + i] = W[(row0 + r) * n + pos];
    }
    subtree_transform<1, true>(T, u, tile, X, nr, false);
#pragma unroll 4
    for (int i = ti; i < ni; i += 64) {
        const int64_t pos = T.in_pos[i0 + i];
        for (int r = tr; r < nr; r += kStageT / 64) W[(row0 + r) * n + pos] = tile[r * X + i];
    }
}

// Row transform of the panel clusters above stage 1 on kRowC columns of W: panel list entry
// u of the tables TP, whose inputs are scaling rows of the panel (at most kRowR); the panel
// root's ns scaling rows also go to the rows u0 .. of U.
__global__ __launch_bounds__(256) void k_rows_panel(double *__restrict__ W, int64_t n, int64_t p0, int64_t u, StageTab TP,
                                                    double *__restrict__ U, int64_t u0, int ns)
{
    extern __shared__ double tile[];
    constexpr int X = kRowC + kPad;
    const int64_t i0 = TP.in_off[u], c0 = (int64_t)blockIdx.x * kRowC;
    const int ni = (int)(TP.in_off[u + 1] - i0), ncol = (int)min<int64_t>(kRowC, n - c0);
    const int cc = threadIdx.x % kRowC, ii = threadIdx.x / kRowC;
    for (int i = ii; i < ni; i += 256 / kRowC)
        if (cc < ncol) tile[i * X + cc] = W[(TP.in_pos[i0 + i] - p0) * n + c0 + cc];
    subtree_transform<1, false>(TP, u, tile, X, ncol, false);
    for (int i = ii; i < ni; i += 256 / kRowC)
        if (cc < ncol) W[(TP.in_pos[i0 + i] - p0) * n + c0 + cc] = tile[i * X + cc];
    const ClusterRec root = TP.rec[TP.lv_start[TP.lv_off[u + 1] - 1] - 1];   // the last cluster of the list
    for (int k = ii; k < ns; k += 256 / kRowC)
        if (cc < ncol) U[(u0 + k) * n + c0 + cc] = tile[root(k) * X + cc];
}

// The panel root's scaling rows (slots sl[0 .. k)) to the rows u0 .. of U.
__global__ void k_scaling_rows(double *__restrict__ U, const double *__restrict__ W, const int64_t *__restrict__ sl,
                               int k, int64_t u0, int64_t n, int64_t p0)
{
    for (int r = 0; r < k; ++r)
        for (int64_t q = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; q < n; q += (int64_t)gridDim.x * blockDim.x)
            U[(u0 + r) * n + q] = W[(sl[r] - p0) * n + q];
}

// One stage of the fast samplet transform of r vectors, 16 at a time: subtree
// sub0 + blockIdx.x.  Input i of a subtree has the slot in_pos[i] and the final place
// out_pos[i] in basis order, or -1 when it is a scaling coefficient that the next stage
// takes over (through the work array W, indexed by slot).  Forward: stage 1 reads the
// points (through the tree's permutation), later stages W; results go to their final
// place in Y or to W.  Inverse (root first): inputs come from X at their place in basis
// order or from W; results go to W, those of stage 1 to the points in Y.
template <bool INV>
__global__ __launch_bounds__(kStageT) void k_fst_stage(const double *__restrict__ X, double *__restrict__ Y,
                                                   double *__restrict__ W, int64_t r, int64_t n, int64_t sub0, int first,
                                                   const int64_t *__restrict__ perm, const int64_t *__restrict__ out_pos,
                                                   StageTab T)
{
    extern __shared__ double tile[];
    const int64_t u = sub0 + blockIdx.x, i0 = T.in_off[u], row0 = (int64_t)blockIdx.y * 16;
    const int ni = (int)(T.in_off[u + 1] - i0), S = ni + kPad, nr = (int)min<int64_t>(16, r - row0);
    // lanes over the inputs, groups of threads over the vectors
    const int tw = 64, ti = threadIdx.x % tw, tr = threadIdx.x / tw, nt = blockDim.x / tw;
    for (int i = ti; i < ni; i += tw) {
        const int64_t pos = T.in_pos[i0 + i], op = out_pos[i0 + i];
        const double *src = INV ? (op >= 0 ? X + op : W + pos) : first ? X + perm[pos] : W + pos;
        for (int j = tr; j < nr; j += nt) tile[j * S + i] = src[(row0 + j) * n];
    }
    subtree_transform<1, true>(T, u, tile, S, nr, INV);
    for (int i = ti; i < ni; i += tw) {
        const int64_t pos = T.in_pos[i0 + i], op = out_pos[i0 + i];
        double *dst = INV ? (first ? Y + perm[pos] : W + pos) : (op >= 0 ? Y + op : W + pos);
        for (int j = tr; j < nr; j += nt) dst[(row0 + j) * n] = tile[j * S + i];
    }
}

// The row transform below keeps Q (m x m) and the inputs of its 64 lanes (m x 64) in
// dynamic LDS sized by the largest cluster of the launch, mmax, so that several
// workgroups share a CU.
__host__ __device__ constexpr size_t tr_lds_bytes(int mmax) { return (size_t)(mmax * mmax + 64 * mmax) * sizeof(double); }

// Row transform: block (cluster list entry, 64 columns); the cluster's input rows
// are R[(rowlist[i] - base) * n + q].
__global__ __launch_bounds__(64) void k_rowtr(double *__restrict__ R, int64_t n, int64_t base,
                                              const int32_t *__restrict__ clist, const int32_t *__restrict__ nin,
                                              const int64_t *__restrict__ qoff, const double *__restrict__ qmat,
                                              const int64_t *__restrict__ rloff, const int64_t *__restrict__ rlist,
                                              int mmax)
{
    extern __shared__ double tr_smem[];
    double *sQ = tr_smem, *sIn = tr_smem + mmax * mmax;
    const int c = clist[blockIdx.x];
    const int m = nin[c];
    const double *Q = qmat + qoff[c];
    for (int e = threadIdx.x; e < m * m; e += 64) sQ[e] = Q[e];
    const int64_t *rl = rlist + rloff[c];
    const int64_t q = (int64_t)blockIdx.y * 64 + threadIdx.x;
    __syncthreads();
    if (q >= n) return;
    for (int i = 0; i < m; ++i) sIn[i * 64 + threadIdx.x] = R[(rl[i] - base) * n + q];
    for (int k = 0; k < m; ++k) {
        double acc = 0.0;
        for (int i = 0; i < m; ++i) acc = fma(sQ[k * m + i], sIn[i * 64 + threadIdx.x], acc);
        R[(rl[k] - base) * n + q] = acc;
    }
}

// Samplet rows of block rows -> tiles.  Element (i, j) of tile (r, c) is the value of
// basis row cstart[r] + i (output kb[r] + i of cluster r) at basis column cstart[c] + j.
// Workgroups (x, y): block row clist[x], every gridDim.y-th of its tiles; a tile is read along
// its rows and written along its columns, through LDS.
__global__ __launch_bounds__(64) void k_extract(double *__restrict__ vals, const double *__restrict__ R, int64_t n,
                                                int64_t base, const int32_t *__restrict__ clist,
                                                const int64_t *__restrict__ blk_rp, const int32_t *__restrict__ tile_col,
                                                const int64_t *__restrict__ tile_off, const int32_t *__restrict__ nfun,
                                                const int64_t *__restrict__ cstart, const int32_t *__restrict__ kb,
                                                const int64_t *__restrict__ rloff, const int64_t *__restrict__ rlist,
                                                const int64_t *__restrict__ slot_of_basis, const uint8_t *__restrict__ keep)
{
    __shared__ double tile[spm::kMaxFun * (spm::kMaxFun + 1)];
    const int r = clist[blockIdx.x], nr = nfun[r];
    if (nr == 0) return;
    const int64_t *rows = rlist + rloff[r] + kb[r];
    const int lane = threadIdx.x;
    for (int64_t t = blk_rp[r] + blockIdx.y; t < blk_rp[r + 1]; t += gridDim.y) {
        const int c = tile_col[t], ncl = nfun[c], ne = nr * ncl;
        const int64_t off = tile_off[t];
        const float rc = 1.0f / (float)ncl, rr = 1.0f / (float)nr;
        const int64_t slot = lane < ncl ? slot_of_basis[cstart[c] + lane] : 0;
        const int64_t row = lane < nr ? rows[lane] - base : 0;
        for (int e0 = 0; e0 < ne; e0 += 64) {          // e < 1024: (e + 1/2) / n in float is exact enough
            const int e = e0 + lane;
            const int i = (int)(((float)e + 0.5f) * rc), j = e - i * ncl;
            const int64_t rw = __shfl(row, i & 63), sl = __shfl(slot, j);
            if (e < ne) tile[i * (spm::kMaxFun + 1) + j] = R[rw * n + sl];
        }
        __syncthreads();
        for (int e = lane; e < ne; e += 64) {
            const int j = (int)(((float)e + 0.5f) * rr), i = e - j * nr;
            vals[off + e] = (keep && !keep[off + e]) ? 0.0 : tile[i * (spm::kMaxFun + 1) + j];
        }
        __syncthreads();
    }
}

double fact(int k)
{
    double f = 1.0;
    for (int i = 2; i <= k; ++i) f *= i;
    return f;
}

// Lets a kernel use more than 64 KiB of dynamic LDS (set once per device).
int allow_lds(const void *k)
{
    static std::mutex mu;
    static std::set<std::pair<int, const void *>> ready;   // (device, kernel)
    int dev = 0;
    SPM_HIP(hipGetDevice(&dev));
    std::lock_guard<std::mutex> lock(mu);
    if (!ready.count({dev, k})) {
        SPM_HIP(hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024));
        ready.insert({dev, k});
    }
    return SPM_OK;
}

// Tables in one device block: host vectors (which stay as they are until the upload), the
// small ones collected into one copy, and space for what the device fills itself.
struct Uploader {
    struct Part {
        void **dst;                                    // device pointer to set
        const void *src;                               // host data, or null
        size_t bytes, off;
    };
    std::vector<Part> parts;
    template <typename T>
    void add(const T *&dst, const std::vector<T> &v) { parts.push_back({(void **)&dst, v.data(), v.size() * sizeof(T), 0}); }
    template <typename T>
    void space(const T *&dst, int64_t n) { parts.push_back({(void **)&dst, nullptr, (size_t)n * sizeof(T), 0}); }
    int upload(void *&block, const char *name)
    {
        constexpr size_t kSmall = 64 * 1024;
        std::stable_partition(parts.begin(), parts.end(), [](const Part &p) { return p.src && p.bytes <= kSmall; });
        size_t total = 0;
        std::vector<char> small;
        for (Part &p : parts) {
            p.off = total;
            total += (p.bytes + 255) & ~(size_t)255;
            if (p.src && p.bytes <= kSmall) {
                small.resize(total);
                if (p.bytes) std::memcpy(small.data() + p.off, p.src, p.bytes);
            }
        }
        if (hipMalloc(&block, std::max<size_t>(256, total)) != hipSuccess) {
            block = nullptr;
            return fail(SPM_ENOMEM, std::string(name) + ": device tables");
        }
        char *const d = static_cast<char *>(block);
        hipError_t e = small.empty() ? hipSuccess : hipMemcpy(d, small.data(), small.size(), hipMemcpyHostToDevice);
        for (const Part &p : parts)
            if (e == hipSuccess && p.src && p.bytes > kSmall) e = hipMemcpy(d + p.off, p.src, p.bytes, hipMemcpyHostToDevice);
        if (e != hipSuccess) {
            (void)hipFree(block);
            block = nullptr;
            return fail(SPM_EHIP, std::string(name) + ": copy of the device tables failed");
        }
        for (const Part &p : parts) *p.dst = d + p.off;
        return SPM_OK;
    }
};

// Subtrees with their inputs and levels, under construction.
struct SubTables {
    std::vector<int64_t> in_off{0}, lv_off{0}, lv_start, in_pos;
    std::vector<ClusterRec> rec;
    const std::vector<int64_t> &foff;                 // fragments of every cluster's matrix
    explicit SubTables(const std::vector<int64_t> &f) : foff(f) {}
    // adds the subtree of clusters `members` with the given input slots; index_of (one entry
    // per slot of the tree) is scratch
    void add(const spm_tree_s *t, std::vector<int32_t> &members, const std::vector<int64_t> &inputs,
             std::vector<int32_t> &index_of)
    {
        std::sort(members.begin(), members.end(), [&](int32_t a, int32_t b) {
            return t->level[a] != t->level[b] ? t->level[a] > t->level[b] : a < b;
        });
        for (size_t i = 0; i < inputs.size(); ++i) index_of[inputs[i]] = (int32_t)i;
        int lev = -1;
        for (int32_t c : members) {
            if (t->level[c] != lev) lv_start.push_back((int64_t)rec.size());
            lev = t->level[c];
            const int m = t->nin[c];
            auto at = [&](int k) { return index_of[t->slots[t->slotoff[c] + k]]; };
            const int first = t->son0[c] < 0 ? m : t->nscal[t->son0[c]];   // inputs of the first run
            ClusterRec R{foff[c], m, first, m > 0 ? at(0) : 0, first < m ? at(first) : 0};
            if (first > 0 && R.base1 == R.base0 + first) R.n0 = m;         // the second continues it
            if (first == 0) R = {foff[c], m, m, R.base1, 0};
            rec.push_back(R);
        }
        lv_start.push_back((int64_t)rec.size());
        lv_off.push_back((int64_t)lv_start.size());
        in_pos.insert(in_pos.end(), inputs.begin(), inputs.end());
        in_off.push_back((int64_t)in_pos.size());
    }
    void put(Uploader &u, StageTab &T)
    {
        u.add(T.in_off, in_off); u.add(T.lv_off, lv_off); u.add(T.lv_start, lv_start);
        u.add(T.in_pos, in_pos); u.add(T.rec, rec);
    }
};

}  // namespace

// One device's copies of a tree's transform tables, kept with the tree (it is immutable):
// the stages from the first fast samplet transform or construction there, the inverse
// matrices from the first transform of either direction (later ones allocate no tables),
// the panels from the first construction.
struct spm::TreeDevice {
    bool have_stages = false, have_inverse = false, have_panels = false;
    void *block = nullptr, *iblock = nullptr, *pblock = nullptr;
    // stages
    StageTab T{}, TP{};
    const double *q = nullptr, *finv = nullptr;        // matrices; fragments of the inverse transforms
    std::vector<int64_t> foff;
    const int64_t *out_pos = nullptr, *perm = nullptr, *qoff = nullptr, *d_foff = nullptr;   // d_foff: foff on the device
    const int32_t *nin = nullptr;
    struct Stage {
        int64_t sub0, count;
        int max_in;
    };
    std::vector<Stage> stages;
    std::vector<int32_t> sub_root;                    // root cluster of every subtree
    // panels
    const double *pts = nullptr;
    const int64_t *sob = nullptr, *slots = nullptr, *sloff = nullptr;
    const int32_t *clist = nullptr, *kb = nullptr;
    const int64_t *urloff = nullptr, *urows = nullptr;
    struct Panel {
        int32_t root;
        int64_t sub0, nsub;                           // stage-1 subtrees of its rows
        int64_t members, nmembers;                    // its clusters in clist
        int rows_in;                                  // scaling rows of its upper clusters
        std::vector<std::pair<int64_t, int64_t>> lv;  // upper clusters by level in clist, deepest first
        int64_t u0;                                   // first scaling row in U
    };
    std::vector<Panel> panels;
    std::vector<std::pair<int64_t, int64_t>> lvl_up;  // clusters above the panels by level in clist, deepest first
    std::vector<int> mmax_up;
    std::vector<std::vector<int>> mmax_panel;
    int64_t nu = 0, maxrows = 0;
    ~TreeDevice()
    {
        for (void *b : {block, iblock, pblock})
            if (b) (void)hipFree(b);
    }
    int need_stages(const spm_tree_s *t, const char *name);
    int need_inverse(const spm_tree_s *t, const char *name);
    int need_panels(const spm_tree_s *t, const char *name);
    int fragments(const spm_tree_s *t, const double *f, bool inv, const char *name) const;
};

spm::TreeTables::~TreeTables()
{
    for (auto &e : by_device) delete e.second;
}

// Fills f with the fragments of every cluster (k_fragments), complete on return.
int spm::TreeDevice::fragments(const spm_tree_s *t, const double *f, bool inv, const char *name) const
{
    hipLaunchKernelGGL(k_fragments, dim3((unsigned)t->nc), dim3(256), 0, nullptr, nin, qoff, d_foff, q, const_cast<double *>(f), inv);
    if (hipGetLastError() != hipSuccess || hipStreamSynchronize(nullptr) != hipSuccess)
        return fail(SPM_EHIP, std::string(name) + ": the device tables could not be formed");
    return SPM_OK;
}

int spm::TreeDevice::need_inverse(const spm_tree_s *t, const char *name)
{
    if (have_inverse) return SPM_OK;
    Uploader up;
    up.space(finv, foff.back());
    int rc = iblock ? SPM_OK : up.upload(iblock, name);
    if (rc == SPM_OK) rc = fragments(t, finv, true, name);
    have_inverse = rc == SPM_OK;
    return rc;
}

int spm::TreeDevice::need_stages(const spm_tree_s *t, const char *name)
{
    if (have_stages) return SPM_OK;
    const int nc = t->nc;
    const int64_t n = t->n;
    foff.assign(nc + 1, 0);
    for (int c = 0; c < nc; ++c) foff[c + 1] = foff[c] + frag_index(t->nin[c], (t->nin[c] + 15) / 16, 0);
    SubTables st(foff);
    std::vector<int32_t> index_of(n);
    std::vector<int64_t> bos(n);                       // basis index of the coefficient in a slot
    for (int c = 0; c < nc; ++c) {
        const int k0 = c == 0 ? 0 : t->nscal[c];
        for (int k = k0; k < t->nin[c]; ++k) bos[t->slots[t->slotoff[c] + k]] = t->cstart[c] + (k - k0);
    }
    st.rec.reserve(nc);
    st.in_pos.reserve(n + n / 2);
    stages.clear();
    sub_root.clear();
    std::vector<char> covered(nc, 0);                  // in a subtree of an earlier stage
    std::vector<int64_t> outv, width(nc);
    outv.reserve(n + n / 2);
    std::vector<int32_t> members;
    std::vector<int64_t> inputs;
    auto hand_over = [&](int c, int k) {               // the first k inputs of c become inputs of the subtree
        const int64_t *sl = t->slots.data() + t->slotoff[c];
        inputs.insert(inputs.end(), sl, sl + k);
    };
    for (bool done = false; !done;) {
        const bool first = stages.empty();
        // inputs of the subtree rooted at c: its points, or its topmost covered clusters'
        // scaling coefficients (sons are numbered after their father)
        for (int c = nc - 1; c >= 0; --c)
            width[c] = first ? t->psize[c]
                             : covered[c] ? t->nscal[c] : width[t->son0[c]] + width[t->son1[c]];
        Stage S{(int64_t)st.in_off.size() - 1, 0, 0};
        std::vector<int32_t> roots, stack(1, 0);
        while (!stack.empty()) {
            const int c = stack.back();
            stack.pop_back();
            if (width[c] <= (first ? kBlk : kSub) || covered[c] || t->son0[c] < 0) { roots.push_back(c); continue; }
            stack.push_back(t->son1[c]);
            stack.push_back(t->son0[c]);
        }
        for (int32_t root : roots) {
            members.clear();
            inputs.clear();
            stack.assign(1, root);
            while (!stack.empty()) {
                const int c = stack.back();
                stack.pop_back();
                if (covered[c]) {                      // its scaling coefficients
                    hand_over(c, t->nscal[c]);
                    continue;
                }
                members.push_back(c);
                if (t->son0[c] >= 0) { stack.push_back(t->son1[c]); stack.push_back(t->son0[c]); }
                else hand_over(c, t->nin[c]);
            }
            st.add(t, members, inputs, index_of);
            for (int64_t pos : inputs) outv.push_back(bos[pos]);
            if (root != 0)                             // handed on to the next stage
                for (int k = 0; k < t->nscal[root]; ++k)
                    outv[outv.size() - inputs.size() + index_of[t->slots[t->slotoff[root] + k]]] = -1;
            sub_root.push_back(root);
            S.max_in = std::max(S.max_in, (int)inputs.size());
            ++S.count;
        }
        for (int32_t root : roots) {                   // cover the subtrees
            stack.assign(1, root);
            while (!stack.empty()) {
                const int c = stack.back();
                stack.pop_back();
                if (covered[c]) continue;
                covered[c] = 1;
                if (t->son0[c] >= 0) { stack.push_back(t->son1[c]); stack.push_back(t->son0[c]); }
            }
        }
        stages.push_back(S);
        done = roots.size() == 1 && roots[0] == 0;
    }
    Uploader up;
    st.put(up, T);
    up.space(T.f, foff.back());
    up.add(d_foff, foff);
    up.add(nin, t->nin); up.add(qoff, t->qoff); up.add(q, t->qmat);
    up.add(out_pos, outv); up.add(perm, t->perm);
    if (block) (void)hipFree(block);                   // of a call that failed after the copies
    block = nullptr;
    int rc = up.upload(block, name);
    if (rc == SPM_OK) rc = fragments(t, T.f, false, name);
    have_stages = rc == SPM_OK;
    return rc;
}

int spm::TreeDevice::need_panels(const spm_tree_s *t, const char *name)
{
    if (have_panels) return SPM_OK;
    const int nc = t->nc, depth = t->depth;
    const int64_t n = t->n;
    std::vector<std::vector<int32_t>> bylevel(depth + 1);
    for (int c = 0; c < nc; ++c) bylevel[t->level[c]].push_back(c);
    const Stage &S1 = stages[0];
    std::vector<char> blk_root(nc, 0);                 // root of a stage-1 subtree
    for (int64_t u = 0; u < S1.count; ++u) blk_root[sub_root[u]] = 1;

    // Panel level lp: the panel buffer holds the rows of the largest panel root, the
    // upper buffer the scaling rows of all panel roots, both n doubles wide.  Take the
    // level that needs the fewest rows in the two together, among the levels whose
    // panel fits the budget and whose panels are made of whole stage-1 subtrees.
    const double budget = 16.0 * 1024 * 1024 * 1024;  // bytes of one panel
    int lp = -1;
    int64_t best = -1;
    for (int l = 0; l <= depth; ++l) {
        int64_t mx = 0, nup = 0;
        bool whole = true;
        for (int k = 0; k <= l; ++k)
            for (int c : bylevel[k]) {
                if (k < l && t->son0[c] >= 0) continue;
                mx = std::max(mx, t->psize[c]);
                if (c != 0) nup += t->nscal[c];
                whole = whole && (blk_root[c] || t->psize[c] > kBlk);
            }
        if (!whole) break;                             // deeper panels are no larger
        if ((double)mx * n * 8.0 > budget && lp >= 0) continue;
        if (lp < 0 || mx + nup < best || (double)maxrows * n * 8.0 > budget) { best = mx + nup; lp = l; maxrows = mx; }
    }
    std::vector<int32_t> roots;                        // panel roots, in the order of their points
    for (int c = 0; c < nc; ++c)
        if (t->level[c] == lp || (t->level[c] < lp && t->son0[c] < 0)) roots.push_back(c);
    std::sort(roots.begin(), roots.end(), [&](int a, int b) { return t->pstart[a] < t->pstart[b]; });
    // rows of U: panel roots get their scaling rows, upper clusters reuse their sons' rows in place
    std::vector<std::vector<int64_t>> ul(nc);
    std::vector<int32_t> cl;
    panels.clear();
    mmax_panel.clear();
    nu = 0;
    SubTables pt(foff);
    std::vector<int32_t> index_of(n);
    auto level_list = [&](const std::vector<int32_t> &v, std::vector<std::pair<int64_t, int64_t>> &lv,
                          std::vector<int> &mm) {      // v sorted by level, deepest first
        for (size_t i = 0; i < v.size();) {
            size_t j = i;
            int mx = 1;
            while (j < v.size() && t->level[v[j]] == t->level[v[i]]) mx = std::max(mx, t->nin[v[j++]]);
            lv.push_back({(int64_t)cl.size(), (int64_t)(j - i)});
            mm.push_back(mx);
            cl.insert(cl.end(), v.begin() + i, v.begin() + j);
            i = j;
        }
    };
    int64_t sub = 0;
    for (int pr : roots) {
        Panel P;
        P.root = pr;
        P.sub0 = sub;
        while (sub < S1.count && t->pstart[sub_root[sub]] < t->pstart[pr] + t->psize[pr]) ++sub;
        P.nsub = sub - P.sub0;
        std::vector<int32_t> members, upper, stack(1, pr);
        std::vector<char> inside;
        std::vector<int64_t> inputs;
        for (int64_t u = P.sub0; u < sub; ++u)         // the panel's scaling rows
            for (int k = 0; k < t->nscal[sub_root[u]]; ++k)
                inputs.push_back(t->slots[t->slotoff[sub_root[u]] + k]);
        while (!stack.empty()) {
            const int c = stack.back();
            stack.pop_back();
            members.push_back(c);
            if (t->psize[c] > kBlk && t->son0[c] >= 0) upper.push_back(c);
            if (t->son0[c] >= 0) { stack.push_back(t->son0[c]); stack.push_back(t->son1[c]); }
        }
        pt.add(t, upper, inputs, index_of);       // also sorts `upper` deepest first
        P.rows_in = (int)inputs.size();
        mmax_panel.emplace_back();
        level_list(upper, P.lv, mmax_panel.back());
        std::sort(members.begin(), members.end());
        P.members = (int64_t)cl.size();
        P.nmembers = (int64_t)members.size();
        cl.insert(cl.end(), members.begin(), members.end());
        P.u0 = nu;
        if (pr != 0)
            for (int k = 0; k < t->nscal[pr]; ++k) ul[pr].push_back(nu++);
        panels.push_back(std::move(P));
    }
    std::vector<int32_t> above;
    for (int l = lp - 1; l >= 0; --l)
        for (int c : bylevel[l]) {
            if (t->son0[c] < 0) continue;
            const int a = t->son0[c], b = t->son1[c];
            ul[c].insert(ul[c].end(), ul[a].begin(), ul[a].begin() + t->nscal[a]);
            ul[c].insert(ul[c].end(), ul[b].begin(), ul[b].begin() + t->nscal[b]);
            above.push_back(c);
        }
    lvl_up.clear();
    mmax_up.clear();
    level_list(above, lvl_up, mmax_up);
    std::vector<int64_t> urloffv(nc), urowsv;
    for (int c = 0; c < nc; ++c) {
        urloffv[c] = (int64_t)urowsv.size();
        urowsv.insert(urowsv.end(), ul[c].begin(), ul[c].end());
    }
    std::vector<int32_t> kbv(nc);
    std::vector<int64_t> sobv(n);                      // slot of a basis function's coefficient
    for (int c = 0; c < nc; ++c) {
        kbv[c] = c == 0 ? 0 : t->nscal[c];
        for (int k = kbv[c]; k < t->nin[c]; ++k) sobv[t->cstart[c] + (k - kbv[c])] = t->slots[t->slotoff[c] + k];
    }
    TP = T;
    Uploader up;
    pt.put(up, TP);
    up.add(sob, sobv); up.add(kb, kbv); up.add(sloff, t->slotoff); up.add(slots, t->slots);
    up.add(pts, t->pts); up.add(clist, cl); up.add(urloff, urloffv); up.add(urows, urowsv);
    const int rc = up.upload(pblock, name);
    have_panels = rc == SPM_OK;
    return rc;
}

// The tree's tables on the current device (stages, and the construction's panels or the
// transforms' inverse matrices), uploaded once with synchronous copies.
enum TreeNeed { TREE_FORWARD, TREE_INVERSE, TREE_PANELS };
static int tree_tables(spm_tree t, TreeNeed need, hipStream_t s, const spm::TreeDevice **out, const char *name)
{
    int dev = 0, st;
    SPM_HIP(hipGetDevice(&dev));
    hipStreamCaptureStatus cap = hipStreamCaptureStatusNone;
    if (need == TREE_FORWARD && hipStreamIsCapturing(s, &cap) != hipSuccess) {   // (another stream's, on the null stream)
        (void)hipGetLastError();
        cap = hipStreamCaptureStatusActive;
    }
    std::lock_guard<std::mutex> lock(t->tables.mu);
    try {
        spm::TreeDevice *&D = t->tables.by_device[dev];
        if (!D) D = new spm::TreeDevice;
        if ((st = D->need_stages(t, name))) return st;
        if (need == TREE_INVERSE && (st = D->need_inverse(t, name))) return st;
        // a forward transform goes without them where they find no memory or the stream is being
        // captured (a construction may have left the stages); an inverse tries again
        if (need == TREE_FORWARD && cap == hipStreamCaptureStatusNone && D->need_inverse(t, name)) (void)hipGetLastError();
        if (need == TREE_PANELS && (st = D->need_panels(t, name))) return st;
        *out = D;
    } catch (const std::bad_alloc &) {
        return fail(SPM_ENOMEM, std::string(name) + ": host allocation");
    }
    return SPM_OK;
}

namespace {

// Stream-ordered device memory, freed in stream order.  The pool keeps what is freed until
// the stream is next synchronised, and no longer.
struct StreamBuf {
    double *p = nullptr;
    hipStream_t s;
    explicit StreamBuf(hipStream_t st) : s(st) {}
    bool get(size_t bytes)
    {
        if (hipMallocAsync((void **)&p, bytes, s) == hipSuccess) return true;
        p = nullptr;
        return false;
    }
    void free()
    {
        if (p) (void)hipFreeAsync(p, s);
        p = nullptr;
    }
    ~StreamBuf() { free(); }
};

// The panel buffers of a construction: however it ends, they have been given back when it returns.
struct PanelBufs {
    hipStream_t s;
    StreamBuf W, U;
    explicit PanelBufs(hipStream_t st) : s(st), W(st), U(st) {}
    hipError_t finish()
    {
        W.free();
        U.free();
        return hipStreamSynchronize(s);
    }
    ~PanelBufs() { if (W.p || U.p) (void)finish(); }
};

}  // namespace

extern "C" int spm_kernel_compress(spm_pattern p, spm_tree t, int32_t mp, double ell, double scale, int32_t deriv,
                                   double *vals, void *stream)
{
    if (!p || !t || !vals) return fail(SPM_EINVAL, "spm_kernel_compress: null pointer");
    SPM_NEED_DEVICE(p, "spm_kernel_compress");
    if (mp < 0 || mp > 3 || !(ell > 0.0)) return fail(SPM_EINVAL, "spm_kernel_compress: bad kernel parameters");
    if (p->n != t->n || p->nc != t->nc || p->cstart != t->cstart)
        return fail(SPM_EINVAL, "spm_kernel_compress: pattern was not built on this tree's clusters");
    const int nc = t->nc, d = t->d;
    const int64_t n = t->n;
    for (int c = 0; c < nc; ++c)
        if (t->nin[c] > kMaxIn) return fail(SPM_EUNSUPPORTED, "spm_kernel_compress: more than 64 inputs in one cluster");
    hipStream_t s = (hipStream_t)stream;

    KParams kp;
    kp.p = mp;
    for (int k = 0; k < 4; ++k) kp.c[k] = 0.0;
    for (int q = 0; q <= mp; ++q) {
        const int k = mp - q;
        kp.c[k] += fact(mp) / fact(2 * mp) * fact(mp + q) / (fact(q) * fact(mp - q)) * std::ldexp(1.0, k);
    }
    kp.sfac = std::sqrt(2.0 * mp + 1.0) / ell;
    kp.ell = ell;
    kp.scale = scale;
    kp.deriv = deriv ? 1 : 0;

    const spm::TreeDevice *D;
    int st;
    if ((st = tree_tables(t, TREE_PANELS, s, &D, "spm_kernel_compress"))) return st;
    PanelBufs bufs(s);
    StreamBuf &W = bufs.W, &U = bufs.U;
    if (!W.get((size_t)D->maxrows * n * sizeof(double))) return fail(SPM_ENOMEM, "spm_kernel_compress: panel buffer");
    if (D->nu > 0 && !U.get((size_t)D->nu * n * sizeof(double))) return fail(SPM_ENOMEM, "spm_kernel_compress: upper buffer");
    if ((st = allow_lds((const void *)k_rows_panel))) return st;

    auto extract = [&](double *R, int64_t base, int64_t c0, int64_t cnt, const int64_t *rloff, const int64_t *rl) -> int {
        if (cnt == 0) return SPM_OK;
        const unsigned gy = (unsigned)std::max<int64_t>(1, std::min<int64_t>(512, 16384 / cnt));
        hipLaunchKernelGGL(k_extract, dim3((unsigned)cnt, gy), dim3(64), 0, s, vals, R, n, base, D->clist + c0,
                           p->d_blk_rp.ptr, p->d_tile_col.ptr, p->d_tile_off.ptr, p->d_nfun.ptr, p->d_cstart.ptr, D->kb,
                           rloff, rl, D->sob, p->d_keep.ptr);
        SPM_HIP(hipGetLastError());
        return SPM_OK;
    };
    auto rowtr = [&](double *R, int64_t base, std::pair<int64_t, int64_t> lv, int mx, const int64_t *rloff,
                     const int64_t *rl) {
        hipLaunchKernelGGL(k_rowtr, dim3((unsigned)lv.second, (unsigned)((n + 63) / 64)), dim3(64), tr_lds_bytes(mx), s,
                           R, n, base, D->clist + lv.first, D->nin, D->qoff, D->q, rloff, rl, mx);
    };

    // progress on stderr (SPM_PROGRESS set): the construction is O(n^2) and runs for
    // many seconds at a million points
    const bool progress = std::getenv("SPM_PROGRESS") != nullptr;
    const size_t tick = std::max<size_t>(1, D->panels.size() / 10);
    const auto &stages = D->stages;
    for (size_t pi = 0; pi < D->panels.size(); ++pi) {
        const auto &P = D->panels[pi];
        if (progress && pi > 0 && pi % tick == 0) {
            SPM_HIP(hipStreamSynchronize(s));
            std::fprintf(stderr, "[spm] kernel_compress: %zu of %zu panels\n", pi, D->panels.size());
        }
        const int64_t p0 = t->pstart[P.root], rows = t->psize[P.root];
        const dim3 ge((unsigned)stages[0].count, (unsigned)P.nsub);
        const bool both = stages.size() == 1;
        switch (mp) {
        case 0: hipLaunchKernelGGL(k_eval_block<0>, ge, dim3(256), 0, s, W.p, D->pts, d, p0, n, P.sub0, kp, D->T, both); break;
        case 1: hipLaunchKernelGGL(k_eval_block<1>, ge, dim3(256), 0, s, W.p, D->pts, d, p0, n, P.sub0, kp, D->T, both); break;
        case 2: hipLaunchKernelGGL(k_eval_block<2>, ge, dim3(256), 0, s, W.p, D->pts, d, p0, n, P.sub0, kp, D->T, both); break;
        default: hipLaunchKernelGGL(k_eval_block<3>, ge, dim3(256), 0, s, W.p, D->pts, d, p0, n, P.sub0, kp, D->T, both); break;
        }
        for (size_t j = 1; j < stages.size(); ++j)
            hipLaunchKernelGGL(k_cols_stage, dim3((unsigned)stages[j].count, (unsigned)((rows + 15) / 16)), dim3(kStageT),
                               16 * (stages[j].max_in + kPad) * sizeof(double), s, W.p, rows, n, stages[j].sub0, D->T);
        if (!both)
            hipLaunchKernelGGL(k_rows_block, dim3((unsigned)((n + kBlk - 1) / kBlk), (unsigned)P.nsub), dim3(256), 0, s, W.p,
                               p0, n, P.sub0, D->T);
        if (!P.lv.empty()) {
            if (P.rows_in <= kRowR)
                hipLaunchKernelGGL(k_rows_panel, dim3((unsigned)((n + kRowC - 1) / kRowC)), dim3(256),
                                   (size_t)P.rows_in * (kRowC + kPad) * sizeof(double), s, W.p, n, p0, (int64_t)pi, D->TP,
                                   U.p, P.u0, P.root != 0 ? t->nscal[P.root] : 0);
            else
                for (size_t l = 0; l < P.lv.size(); ++l)
                    rowtr(W.p, p0, P.lv[l], D->mmax_panel[pi][l], D->sloff, D->slots);
        }
        SPM_HIP(hipGetLastError());
        if ((st = extract(W.p, p0, P.members, P.nmembers, D->sloff, D->slots))) return st;
        if (P.root != 0 && (P.lv.empty() || P.rows_in > kRowR))
            hipLaunchKernelGGL(k_scaling_rows, dim3((unsigned)std::min<int64_t>((n + 255) / 256, 4096)), dim3(256), 0, s,
                               U.p, W.p, D->slots + t->slotoff[P.root], t->nscal[P.root], P.u0, n, p0);
    }
    for (size_t i = 0; i < D->lvl_up.size(); ++i) {
        rowtr(U.p, 0, D->lvl_up[i], D->mmax_up[i], D->urloff, D->urows);
        SPM_HIP(hipGetLastError());
        if ((st = extract(U.p, 0, D->lvl_up[i].first, D->lvl_up[i].second, D->urloff, D->urows))) return st;
    }
    SPM_HIP(bufs.finish());
    return SPM_OK;
}

// Fast samplet transform of r vectors (Section 3.2): Y = T X with X in the points'
// original order and Y in basis order, or the inverse X = T^T Y, one launch per stage of
// the tree (three at 131072 points with four moments, four at a million with six; one per
// level, plus the permutations, was bound by the launches).
extern "C" int spm_fst(spm_tree t, const double *X, int32_t r, double *Y, int32_t inverse, void *stream)
{
    if (!t) return fail(SPM_EINVAL, "spm_fst: null tree");
    if (r < 0) return fail(SPM_EINVAL, "spm_fst: negative vector count");
    const int64_t n = t->n, total = (int64_t)r * n;
    if (r == 0 || n == 0) return SPM_OK;                     // X and Y may then be null
    if (!X || !Y) return fail(SPM_EINVAL, "spm_fst: null pointer");
    {
        const char *x0 = reinterpret_cast<const char *>(X), *y0 = reinterpret_cast<const char *>(Y);
        const size_t b = (size_t)total * sizeof(double);
        if (x0 < y0 + b && y0 < x0 + b) return fail(SPM_EINVAL, "spm_fst: X and Y overlap");
    }
    const int nc = t->nc;
    for (int c = 0; c < nc; ++c)
        if (t->nin[c] > kMaxIn) return fail(SPM_EUNSUPPORTED, "spm_fst: more than 64 inputs in one cluster");
    hipStream_t s = (hipStream_t)stream;
    const spm::TreeDevice *D;
    int st;
    if ((st = tree_tables(t, inverse ? TREE_INVERSE : TREE_FORWARD, s, &D, "spm_fst"))) return st;
    StreamBuf W(s);                                    // coefficients between stages, by slot
    if (D->stages.size() > 1 && !W.get((size_t)total * sizeof(double))) return fail(SPM_ENOMEM, "spm_fst: work buffer");
    const int ns = (int)D->stages.size();
    StageTab T = D->T;
    if (inverse) T.f = D->finv;
    for (int i = 0; i < ns; ++i) {
        const int j = inverse ? ns - 1 - i : i;
        const auto &S = D->stages[j];
        const dim3 g((unsigned)S.count, (unsigned)((r + 15) / 16));
        const size_t lds = 16 * (S.max_in + kPad) * sizeof(double);
        if (inverse)
            hipLaunchKernelGGL(k_fst_stage<true>, g, dim3(j == 0 ? 256 : kStageT), lds, s, X, Y, W.p, (int64_t)r, n, S.sub0, j == 0, D->perm,
                               D->out_pos, T);
        else
            hipLaunchKernelGGL(k_fst_stage<false>, g, dim3(j == 0 ? 256 : kStageT), lds, s, X, Y, W.p, (int64_t)r, n, S.sub0, j == 0, D->perm,
                               D->out_pos, T);
    }
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return fail(SPM_EHIP, std::string("spm_fst: launch failed: ") + hipGetErrorString(e));
    return SPM_OK;
}
