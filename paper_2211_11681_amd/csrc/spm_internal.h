// Internal declarations shared by the host and device translation units of libspm.
#pragma once

#include <hip/hip_runtime.h>
#include <sys/mman.h>

#include <cstdint>
#include <cstdlib>
#include <map>
#include <memory>
#include <mutex>
#include <new>
#include <string>
#include <utility>
#include <vector>

#include "../../include/spm.h"

namespace spm {

constexpr int kMaxFun = 32;   // largest number of basis functions per cluster the kernels take
constexpr int64_t kQuadEntries = int64_t(1) << 29;   // largest total of the quads' middle lists (4 GB)
// Fewest quads: two per workgroup the chip holds (256 CUs x 8).  Below, a quad's longer chain
// costs more than its fewer loads give.  Products in ms, units / quads: 289 quads (sphere,
// N = 4096) 0.641 / 0.714, 1071 (cube, 8000) 7.55 / 7.60, 2834 (square, 8000) 3.11 / 3.16,
// 4011 (cube, 12000) 14.1 / 13.4, 9703 (square, 4096) 0.51 / 0.47, 23463 (sphere, 9000)
// 1.27 / 1.11.
constexpr int64_t kQuadMin = 4096;
constexpr int kQuadRows = 32;                        // k rows of a quad's stage
constexpr int kPieceEntries = 2048;   // largest piece of a block row in the S x dense product

int fail(int status, const std::string &msg);   // records msg, returns status

#define SPM_HIP(expr)                                                                       \
    do {                                                                                    \
        hipError_t e_ = (expr);                                                             \
        if (e_ != hipSuccess)                                                               \
            return ::spm::fail(SPM_EHIP, std::string(#expr " failed: ") + hipGetErrorString(e_)); \
    } while (0)

// Compute calls need the pattern's device tables (a planned pattern has host tables only).
#define SPM_NEED_DEVICE(p, name)                                                            \
    do {                                                                                    \
        if (!(p)->uploaded)                                                                 \
            return ::spm::fail(SPM_EINVAL, std::string(name) + ": pattern not uploaded");   \
    } while (0)

// A vector for large tables filled and gathered from by threads: resize leaves the new
// elements unset, and the memory is of huge pages where the system gives them on request
// (the first touch of 1 GB in 4 KB pages takes 136 ms of one thread, 51 ms so).
template <typename T>
struct RawAlloc : std::allocator<T> {
    static constexpr size_t kHuge = size_t(2) << 20, kLarge = 8 * kHuge;
    template <typename U>
    struct rebind { using other = RawAlloc<U>; };
    RawAlloc() = default;
    template <typename U>
    RawAlloc(const RawAlloc<U> &) {}
    T *allocate(size_t n)
    {
        if (n > (SIZE_MAX - kHuge) / sizeof(T)) throw std::bad_array_new_length();
        const size_t bytes = n * sizeof(T);
        if (bytes < kLarge) return std::allocator<T>::allocate(n);
        void *p = std::aligned_alloc(kHuge, (bytes + kHuge - 1) / kHuge * kHuge);
        if (!p) throw std::bad_alloc();
        (void)madvise(p, bytes, MADV_HUGEPAGE);        // advice: small pages otherwise
        return static_cast<T *>(p);
    }
    void deallocate(T *p, size_t n)
    {
        if (n * sizeof(T) < kLarge) std::allocator<T>::deallocate(p, n);
        else std::free(p);
    }
    template <typename U, typename... A>
    void construct(U *p, A &&...a)
    {
        if constexpr (sizeof...(A) == 0) ::new (static_cast<void *>(p)) U;
        else ::new (static_cast<void *>(p)) U(std::forward<A>(a)...);
    }
};
template <typename T>
using RawVec = std::vector<T, RawAlloc<T>>;

// Device copy of a host vector (owned by the pattern / tree handle).
template <typename T>
struct DevBuf {
    T *ptr = nullptr;
    size_t n = 0;
};

// Device copies of a tree's transform tables, per device, uploaded on first use and freed
// with the tree (spm_compress.hip).
struct TreeDevice;
struct TreeTables {
    std::mutex mu;                    // guards the map and the uploads
    std::map<int, TreeDevice *> by_device;
    ~TreeTables();
};

}  // namespace spm

struct spm_tree_s {
    int64_t n = 0;
    int32_t d = 0, leaf = 0, q = 0, m = 0;
    int32_t nc = 0, depth = 0;
    std::vector<double> pts;          // tree order, n x d
    std::vector<int64_t> perm;        // tree position -> original index
    std::vector<int64_t> pstart, psize;
    std::vector<int32_t> level, parent, son0, son1;
    std::vector<double> lo, hi;       // nc x d
    std::vector<int64_t> cstart;      // basis ranges, nc + 1
    // two-scale transforms
    std::vector<int32_t> nin, nscal;  // inputs and scaling functions handed up, per cluster
    std::vector<int64_t> qoff;        // offset of each cluster's Q (nin x nin, column-major)
    std::vector<double> qmat;
    std::vector<int64_t> slotoff;     // offset of each cluster's input slot list
    std::vector<int64_t> slots;       // input slots (tree-order point positions)
    spm::TreeTables tables;
};

struct spm_pattern_s {
    int64_t n = 0, nnz = 0, n_stored = 0, n_tiles = 0;
    int32_t nc = 0;
    double macs = 0.0;
    bool masked = false;              // some tile positions are outside S
    int32_t max_rowlen = 0;           // longest block row (tiles)
    // host structure
    std::vector<int64_t> cstart;      // nc + 1
    std::vector<int32_t> nfun;        // nc
    std::vector<int64_t> blk_rp;      // nc + 1
    std::vector<int32_t> tile_row, tile_col, trans;   // n_tiles
    std::vector<int64_t> tile_off;    // n_tiles + 1
    std::vector<int64_t> diag_pos;    // stored positions of the diagonal entries (of the diagonal tiles), ascending
    std::vector<int64_t> colprefix;   // n_tiles: entries of the tile row before this tile
    std::vector<int64_t> rowbase, rowlen;  // nc: CSR position of the block row's first entry, entries per row
    std::vector<int32_t> diag_tile;   // nc
    // pieces of the block rows for the S x dense product: runs of tiles whose column
    // clusters are consecutive (a dense panel over a contiguous range of basis columns),
    // cut into pieces of whole 16-column chunks and at most kPieceEntries entries
    std::vector<int64_t> pc_rp;       // nc + 1
    std::vector<int64_t> pc_off, pc_g;   // element offset in the value array, first basis column
    std::vector<int32_t> pc_w;        // columns
    std::vector<int32_t> order;       // tile processing order (schedule)
    // grouped schedule of the FP64 product: groups of up to 4 consecutive clusters of
    // one size, and units = pairs of groups holding at least one output tile
    int32_t ng = 0, kmax = 4;         // groups, largest padded cluster size
    std::vector<int32_t> grp_mem;     // ng x 4 member clusters (-1 pads)
    std::vector<int32_t> grp_s, grp_g, grp_R;   // slot size, member count, rows (multiple of 16)
    std::vector<int64_t> gl_rp;       // ng + 1: union lists U(G) = union of the members' block rows
    spm::RawVec<int32_t> gl_mu;       // cluster of each union entry
    spm::RawVec<int32_t> gl_tile;     // entries x 4: tile (member k, mu) or -1
    spm::RawVec<int32_t> unit_gr, unit_gc, unit_out;   // units; unit_out: units x 16 output tiles or -1
    std::vector<int32_t> unit_order;  // unit ids grouped by launch class, costly first
    std::vector<int32_t> unit_order_lv;   // the (1, 1) class for the split-precision product (with levels, even sizes)
    std::vector<int64_t> pair_off;    // units + 1: offsets of each unit's middle-cluster list
    spm::RawVec<int32_t> pair_a, pair_b;   // union-list entries of mu in U(G_r) and U(G_c)
    spm::RawVec<int32_t> gl_nm;       // functions of the cluster of each union entry
    spm::RawVec<int64_t> gl_offd;            // entries x 4: element offset of tile (member, mu), -1 absent
    std::vector<int64_t> stage_off;   // units + 1: stages of each unit
    spm::RawVec<int32_t> stage_first; // first pair of each stage, relative to the unit's pair_off
    struct Launch {
        int32_t rb, cb, waves;
        int32_t smax_r, smax_c;   // largest slot of the row / column groups of the class
        int64_t first, count;
        int64_t out_tiles;        // output tiles of the class
        double exact_macs;        // sum over its output tiles (r, c) of n_r n_c sum_{mu in S_r cap S_c} n_mu
        double padded_macs;       // multiply-adds the kernels issue for it before block skipping
    };
    std::vector<Launch> launches;
    // tree levels of the clusters (optional, given at planning): with them the middle
    // clusters of a unit are ordered level by level and no stage mixes two levels, as the
    // split-precision product scales its operands per row and level
    std::vector<int32_t> clevel;      // nc, or empty
    int32_t nlev = 0;                 // 1 + largest level (0 without levels)
    spm::RawVec<int32_t> gl_nml;      // entries: functions | level << 8 of the entry's cluster
    spm::RawVec<int64_t> gl_offT;     // entries x 4: element offset of tile (mu, member), -1 absent
    // the middle clusters of each unit once more, ordered level by level, and stages of one
    // level each (the split-precision product; the FP64 and FP32 order is kept as it is)
    spm::RawVec<int32_t> pair_a_lv, pair_b_lv;
    std::vector<int64_t> stage_off_lv;    // units + 1
    spm::RawVec<int32_t> stage_first_lv;  // first pair of each stage (relative to the unit's pair_off)
    // Quads of the FP64 product: the units of a single block, two row groups by two column
    // groups at a time, over one list of middle clusters (empty above kQuadEntries entries)
    std::vector<int32_t> quad_unit;   // quads x 4: unit of (row group a, column group b) at 2a + b, or -1
    std::vector<int64_t> quad_off;    // quads + 1: offsets of each quad's middle-cluster list
    spm::RawVec<int32_t> quad_ent;    // x 2: entries of mu in the union lists of the row pair and the column pair
    std::vector<int64_t> quad_stage_off;   // quads + 1
    spm::RawVec<int32_t> quad_stage;  // x 4: first middle cluster; their number | k rows << 8 | groups present << 16;
                                      // bit per k row where a cluster starts; first row taken of the first cluster
    std::vector<int32_t> quad_order;  // launch order
    spm::RawVec<int64_t> pair_offd;   // x 8: as gl_offd for the union lists of the pairs of row groups
    double padded_macs = 0.0;         // multiply-adds the grouped kernel issues (incl. padding)
    bool all_even = false;            // every cluster owns an even number of functions
    bool all_mult4 = false;           // every cluster owns a multiple of 4 functions
    // masked patterns only (entry-level upload)
    std::vector<int64_t> csr_rp;      // n + 1
    std::vector<int32_t> csr_col;
    std::vector<int64_t> csr_pos;     // n_stored: CSR position or -1
    // device copies: every table is carved from one block of device memory, owned by the
    // pattern (uploads that allocate) or by the caller (spm_pattern_upload_workspace)
    bool uploaded = false;
    void *dev_block = nullptr;
    bool owns_block = false;
    std::vector<double> tile_macs;    // n_tiles: exact multiply-adds of each output tile (planning only)
    spm::DevBuf<int64_t> d_cstart, d_blk_rp, d_tile_off, d_colprefix, d_rowbase, d_rowlen, d_csr_pos;
    spm::DevBuf<int64_t> d_pc_rp, d_pc_off, d_pc_g;
    spm::DevBuf<int32_t> d_pc_w;
    spm::DevBuf<int32_t> d_nfun, d_tile_row, d_tile_col, d_trans, d_diag_tile, d_order;
    spm::DevBuf<int32_t> d_grp_mem, d_grp_s, d_grp_g, d_grp_R, d_gl_mu, d_gl_tile, d_unit_gr, d_unit_gc, d_unit_out,
        d_unit_order, d_unit_order_lv;
    spm::DevBuf<int64_t> d_gl_rp, d_pair_off, d_gl_offd, d_stage_off;
    spm::DevBuf<int32_t> d_pair_a, d_pair_b, d_gl_nm, d_stage_first;
    spm::DevBuf<int32_t> d_clevel, d_gl_nml, d_stage_first_lv, d_pair_a_lv, d_pair_b_lv;
    spm::DevBuf<int64_t> d_gl_offT, d_stage_off_lv;
    spm::DevBuf<int32_t> d_quad_unit, d_quad_ent, d_quad_stage, d_quad_order;
    spm::DevBuf<int64_t> d_quad_off, d_quad_stage_off, d_pair_offd;
    spm::DevBuf<uint8_t> d_keep;      // n_stored, masked patterns only
    spm::DevBuf<int64_t> d_diag_pos;
    spm::DevBuf<double> d_partial;    // reduction partials
};

namespace spm {
size_t pattern_device_bytes(const spm_pattern_s *p);
// copies the tables into ws (bytes >= pattern_device_bytes), or into a block it
// allocates when ws is null
int upload_pattern_device(spm_pattern_s *p, void *ws, size_t bytes, hipStream_t s);
void free_pattern_device(spm_pattern_s *p);
}  // namespace spm

namespace spm {
int launch_gemm(spm_pattern_s *p, int prec, const void *A, int ta, const void *B, int tb, void *C, hipStream_t s);
size_t gemm_ws_bytes(spm_pattern_s *p, int prec, int ta, int tb);
int gemm_ws(spm_pattern_s *p, int prec, const void *A, int ta, const void *B, int tb, void *C, void *ws, hipStream_t s);
size_t ws_align(size_t x);
int launch_reduce(spm_pattern_s *p, int op, int prec, const void *x, const void *y, const double *vec, double alpha,
                  int post, double scale, double *out, hipStream_t s);
int launch_axpy(spm_pattern_s *p, int prec, double alpha, const void *X, double beta, void *Y, hipStream_t s);
int launch_convert(spm_pattern_s *p, int pf, const void *X, int pt, void *Y, hipStream_t s);
}  // namespace spm
