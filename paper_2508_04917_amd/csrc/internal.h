// Internal declarations of the ddilu GPU library (gfx950 / CDNA4).
#pragma once

#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdint>
#include <string>
#include <vector>

#include "../../include/ddilu.h"

namespace ddilu {

constexpr int kMaxRowBlocks = 64;   // blocks per row accepted by the reorder
constexpr int kWave = 64;           // CDNA wavefront width
constexpr int kMaxSlots = 3;        // largest per-row block count of the slot layout

// Streaming layout of one triangular sweep.  Positions are the rows of each
// subdomain in sweep order (level by level, ascending local row inside a
// level); subdomain s owns positions [s*S, (s+1)*S).  Everything a sweep
// reads is laid out in that order so one workgroup streams its factor data
// front to back.
struct Sweep {
    uint16_t *prow = nullptr;   // [n] local row of each position
    int32_t *bptr = nullptr;    // [n+1] first block of each position
    uint16_t *bcol = nullptr;   // [nblk] local column of each block
    double *val64 = nullptr;    // [nblk*bb] L blocks (lower) or Uhat (upper)
    float *val32 = nullptr;     // FP32 copy (built on demand)
    double *d64 = nullptr;      // upper only: inv_D per position [n*bb]
    double *uraw = nullptr;     // upper only, built on demand: U blocks without the inv_D scaling [nblk*bb]
    int32_t uraw_ready = 0;     // uraw holds the present factors'
    float *d32 = nullptr;
    int64_t nblk = 0;
    int32_t max_row = 0;        // most blocks of any row in this sweep
    // Slot layout (when every row has at most kMaxSlots blocks): position p
    // owns MB block slots (MB = the handle's slot count; unused slots hold
    // zero blocks) and, in the upper sweep, its inv_D block.  Per position the
    // values are stored as BS runs, run i = row i of every slot block then
    // row i of inv_D, so the BS lanes of a row each read one contiguous run.
    // The address of a block is a function of the position alone, so a sweep
    // can issue its loads without first reading row offsets.
    uint64_t *desc = nullptr;   // [n] local row | column of slot k << 16(k+1); 0xFFFF empty
    double *sval64 = nullptr;   // [n*MB*bb] lower, [n*(MB+1)*bb] upper
    float *sval32 = nullptr;
    int64_t snpos = 0;          // positions of the slot layout (n, or the segmented layout's count)
    // Wave-chunks of the slot layouts: a level's positions in pieces of one
    // wavefront pass (64/bs rows), in sweep order; {first position (relative
    // to the subdomain), level << 8 | positions}.  winfo[s]: subdomain s's
    // first chunk, number of chunks, number of levels.
    int2 *wtab = nullptr;
    int4 *winfo = nullptr;
    // Segmented slot layout (rows of more than kMaxSlots blocks): a row is
    // split into segments at consecutive positions of one wave-chunk.  With MB blocks per
    // segment (dd_ctx::seg): a lower-sweep segment holds MB blocks; in the
    // upper sweep the row's first segment holds MB blocks and inv_D, each
    // continuation MB + 1 blocks, the last one in the inv_D slot.  desc then
    // holds 15-bit fields: local row (a continuation of the upper sweep: the
    // column of its extra block) | continuation flag << 15, columns at
    // 16(k+1) (0x7FFF empty), and, for a row's first segment, its segment
    // count minus one in bits 31, 47 and 63.
    int32_t *gpos = nullptr;    // [nsub+1] first position of each subdomain
    int2 *pmap = nullptr;       // [snpos] row, segment | its count << 8
};

constexpr int kSegMax = 8;  // segments of a row in the segmented layout

// Level sets of one factor, per subdomain.
struct Levels {
    int32_t *lev = nullptr;     // [n] level of each row (reordered numbering)
    int32_t *nlev = nullptr;    // [nsub]
    int32_t *off = nullptr;     // [nsub+1] start of each subdomain in ptr
    int32_t *ptr = nullptr;     // [ptr_len] level offsets relative to the subdomain
    int32_t *rows = nullptr;    // [n] local rows grouped by level
    int32_t ptr_len = 0;
    int32_t max_levels = 0;
};

// Learned interface correction state (faces, features, coefficients, and
// the training workspace).
struct Lic {
    int32_t ready = 0, active = 0;
    int32_t nf = 0;               // faces
    int32_t *fptr = nullptr;      // [n+1] faces of each row (CSR order)
    int32_t *fI = nullptr, *fJ = nullptr, *fq = nullptr;  // [nf] row, column, block position in A
    int32_t *diag = nullptr;      // [n] diagonal block position of each row of A
    // the apply's copy of the faces, rank-major per subdomain (first face of
    // every row, then second faces, ...): records, CSR index, coefficients
    int2 *lrec = nullptr;         // [nf] {local row, J}
    int32_t *lperm = nullptr;     // [nf] CSR face index of each rank-major position
    float *Cr = nullptr;          // [nf*9] C in rank-major order
    int32_t *rb = nullptr;        // [nsub*9] faces of ranks < k of subdomain s at rb[9s + k]
    float *X = nullptr;           // [nf*27] features
    float *C = nullptr;           // [nf*9] coefficients
    float *H1 = nullptr, *H2 = nullptr, *G1 = nullptr, *G2 = nullptr, *dC = nullptr;
    double *wpart = nullptr, *rpart = nullptr;
    double *Z = nullptr, *G = nullptr, *A = nullptr;
    int32_t work_q = 0;
    double *adj_val[2] = {nullptr, nullptr};  // transposed slot streams (U^T lower, L^T + inv_D^T upper)
    int32_t adj_ready = 0;                    // adj_val packed from the current factors
};

// Device scalars of one BiCGSTAB run (all FP64 except the control words).
struct KrylovScalars {
    double rho, alpha, omega, beta;
    double bnorm, rnorm, snorm;
    double tol;                  // rtol * ||b||
    int32_t state;               // 0 running, 1 converged, -5 breakdown, -6 no convergence
    int32_t iters;
    int32_t maxit;
    int32_t half;                // 1 when the solve stopped after a half step
};

}  // namespace ddilu

struct dd_ctx {
    // problem and partition
    int32_t nx = 0, ny = 0, nz = 0, bs = 0;
    int32_t sx = 0, sy = 0, sz = 0;
    int32_t S = 0, nsub = 0;
    int32_t graph = 0;            // labels from the graph partitioner (no geometry: nx = n, sx = S)
    int64_t n = 0, nnzb = 0;
    int32_t *part_id = nullptr, *new2old = nullptr, *old2new = nullptr;
    int32_t *asrc = nullptr;      // [nnzb] input block of each reordered block (for ilu0_refactor)
    int32_t *tsrc = nullptr;      // [nnzt] block of A of each block of the dropped pattern
    // full reordered matrix
    int32_t *aptr = nullptr, *acol = nullptr;
    double *aval = nullptr;
    // dropped pattern and factors
    int64_t nnzt = 0, nlow = 0, nupp = 0;
    int32_t *tptr = nullptr, *tcol = nullptr, *tdiag = nullptr;
    double *lu = nullptr;       // L\U in the dropped pattern (see launch_lu_blocks)
    double *invd = nullptr;     // [n*bb] inv(U_II), reordered row order
    ddilu::Levels lev[2];
    ddilu::Sweep sw[2];
    int32_t *linv = nullptr, *uinv = nullptr;  // [n] lower- and upper-sweep position of each row
    int32_t reach = 0;            // how many positions back a row's lower columns lie at most (k_factor_records)
    int4 *frec = nullptr;         // [2n] factor records of the slot layout (k_factor_records)
    int32_t direct = 0;           // factored by launch_bilu0_slots (frec valid for ilu0_refactor)
    int32_t csr_ready = 0;        // the sweeps' CSR streams are built (variants 1, 2, 4-8; rows neither slot layout holds)
    int32_t factored = 0;
    int32_t patterned = 0;        // drop, levels and streaming layouts built (ilu0_refactor may run)
    int32_t precision = DD_FP64;
    int32_t max_level_width = 0;  // widest level of any subdomain, L or U
    int32_t profile = 0;          // time every apply inside bicgstab_solve
    // events the next apply launch records at its kernel's start and end
    // (set by launch_precond for per-apply timing; tev_used: a slot kernel
    // took them)
    hipEvent_t tev[2] = {nullptr, nullptr};
    hipEvent_t tsolve[2] = {nullptr, nullptr};  // start and end of a solve (created by the first)
    int32_t tev_used = 0;
    int32_t slots = 0;            // MB of the slot layout (0: CSR layout only)
    int32_t seg = 0;              // MB of the segmented slot layout (2 or 3; 0: not built)
    int32_t variant = 0;          // apply kernel: 0 auto, 1 simple, 2 pipelined CSR, 3 slots, 4-8 ablations
    double *hist = nullptr;       // optional residual history (device, caller-owned)
    ddilu::Lic lic;
    int32_t pc_kind = 0;          // preconditioner of bicgstab_solve: 0 DD-ILU0, 1 global ILU0
    // global (undecomposed) ILU0 of the full reordered matrix.  Pattern (kept
    // for the handle's life): rows of each level one after another, host
    // offsets of the levels.  Where every row has at most three blocks a
    // sweep, the factors lie in the slot layout at the decomposed sweeps'
    // positions, columns outside the subdomain numbered after its rows
    // (halo); boxes of one level of the subdomain graph run together.
    int32_t *glev[2] = {nullptr, nullptr};
    int32_t *glist[2] = {nullptr, nullptr};
    std::vector<int32_t> glp[2];
    int32_t *gdiag = nullptr;
    int32_t gpattern = 0;         // the above built
    int32_t gslots = 0;           // slot layout in use (else glu/gf)
    int32_t ghalo = 0;            // most halo rows of a subdomain, either sweep
    int4 *grec = nullptr;         // [3n] factor records, level order
    uint64_t *gdesc[2] = {nullptr, nullptr};
    double *gsval[2] = {nullptr, nullptr};
    int32_t *ghptr[2] = {nullptr, nullptr}, *ghrow[2] = {nullptr, nullptr};  // halo rows of each subdomain
    int32_t *gbox[2] = {nullptr, nullptr};  // subdomains by level of the subdomain graph
    std::vector<int32_t> gbp[2];            // offsets of those levels
    double *glu = nullptr, *ginvd = nullptr, *gf = nullptr;
    int32_t gfactored = 0;
    int32_t hist_len = 0;
    std::vector<hipEvent_t> events;
    // scratch
    int32_t *status = nullptr;  // [32] device status words
    int32_t *scan_tmp = nullptr;
    int64_t scan_tmp_len = 0;
    // Krylov workspace (allocated on first solve)
    double *kv = nullptr;       // kKrylovVectors vectors of n*bs
    double *partials = nullptr; // [8 * spmv_part_stride] per-workgroup partial sums
    int32_t spmv_part_stride = 0;
    int32_t max_row_a = 0;               // most blocks in a row of the full matrix
    int32_t ell_state = 0;               // sliced-ELL copy for the SpMV: 0 not built, 1 ready, -1 not used
    int32_t *ell_col = nullptr;          // [slices][width][rows per wavefront]
    double *ell_val = nullptr;           // the same slots, bs*bs values each
    // per-slice widths (rows of more than kUnroll blocks; null otherwise):
    int32_t *sell_row = nullptr;         // [slices][rows per wavefront] block row, longest first (-1: none)
    int32_t *sell_len = nullptr;         // its length
    int64_t *sell_off = nullptr;         // [slices + 1] first slot run of each slice
    int64_t sell_nslice = 0;             // slices of the copy
    int32_t sell_spp = 0;                // slices per part (part-aligned slices, graphs), 0 otherwise
    int32_t lic_fallback = 1;            // rerun a failed learned solve with plain DD-ILU0
    int32_t fuse = 0;                    // apply + SpMV as one launch inside bicgstab_solve (opt-in)
    int32_t *fdep = nullptr;             // [2 nsub] dependency ranges of the SpMV tiles
    uint32_t *fflag = nullptr;           // [nsub] per-subdomain completion epochs
    unsigned long long *fticket = nullptr;  // workgroup ticket counter
    ddilu::KrylovScalars *ks = nullptr;
    ddilu::KrylovScalars *ks_host = nullptr;  // pinned
    std::vector<void *> allocs;   // the handle's device buffers
    std::vector<void *> retired;  // released ones that queued work may still read
    int device = -1;
    std::string err;

    int fail(int code, const char *fmt, ...);
    hipError_t try_alloc(void **p, size_t bytes);  // for memory the call can do without: no error is recorded
    int alloc_bytes(void **p, size_t bytes);
    // device memory of count elements, recorded for dd_destroy
    template <typename T>
    int alloc(T **p, int64_t count) {
        void *q = nullptr;
        const int rc = alloc_bytes(&q, (size_t)std::max<int64_t>(count, 1) * sizeof(T));
        if (!rc) *p = static_cast<T *>(q);
        return rc;
    }
    // to the pool at the next reclaim(); the pointer is cleared
    template <typename T>
    void release(T *&p) {
        retire(p);
        p = nullptr;
    }
    void retire(void *q);
    void reclaim();  // waits for the device when something was released
    ~dd_ctx();
};

namespace ddilu {

// Every way out of a call that releases buffers gives them back.
struct ReclaimAtExit {
    dd_ctx *h;
    ~ReclaimAtExit() { h->reclaim(); }
};

// device memory kept between handles (pool.hip)
hipError_t pool_alloc(void **out, size_t bytes);
void pool_free(void *q);      // the device must have been idle since q's last use
void pool_trim(int device);   // back to the driver; -1: every device

// exclusive scan of int32 counts: out[0] = 0, out[i+1] = out[i] + in[i];
// returns the total in *total (synchronises the stream).  tmp: scratch of
// at least scan_tmp_elems(n) int32.
int64_t scan_tmp_elems(int64_t n);
hipError_t exclusive_scan(const int32_t *in, int32_t *out, int64_t n, int32_t *tmp,
                          hipStream_t st);

}  // namespace ddilu

// kernel launchers implemented in the .hip files
namespace ddilu {
hipError_t launch_partition(dd_ctx *h, hipStream_t st);
// labels, new2old and old2new of a graph without geometry (recursive BFS
// bisection into parts of h->S vertices); DD_OK or an error code
int graph_partition(dd_ctx *h, const int32_t *ptr, const int32_t *col, hipStream_t st);
hipError_t launch_check_rows(int64_t n, int64_t nnzb, const int32_t *ptr, const int32_t *col, int32_t *status,
                             hipStream_t st);
hipError_t launch_row_len(dd_ctx *h, const int32_t *ptr, int32_t *len, hipStream_t st);
hipError_t launch_reorder_rows(dd_ctx *h, const int32_t *ptr, const int32_t *col, int32_t *src, hipStream_t st);
hipError_t launch_drop_count(dd_ctx *h, int32_t *tbeg, int32_t *tlen, hipStream_t st);
hipError_t launch_drop_rows(dd_ctx *h, const int32_t *tbeg, int32_t *tsrc, hipStream_t st);
// both sweeps' level sets; stats (zeroed, 8 words): most blocks of a row, most
// levels, (by launch_level_lists) the widest level, blocks: [0,1], [2,3], [4], [6,7]
hipError_t launch_level_sets(dd_ctx *h, int32_t *stats, hipStream_t st);
hipError_t launch_plus_one(int64_t m, const int32_t *in, int32_t *out, hipStream_t st);
hipError_t launch_level_lists(dd_ctx *h, int32_t *stats, hipStream_t st);
hipError_t launch_bilu0(dd_ctx *h, hipStream_t st);
// slot descriptors and factor records; stats (zeroed): [0] raised where
// launch_bilu0_slots does not apply, [1] reach (see k_factor_records)
hipError_t launch_slot_records(dd_ctx *h, int32_t *stats, hipStream_t st);
hipError_t launch_bilu0_slots(dd_ctx *h, hipStream_t st);
hipError_t launch_pack_count(dd_ctx *h, int which, int32_t *cnt, hipStream_t st);
hipError_t launch_lu_blocks(dd_ctx *h, hipStream_t st);  // lu, before it is read
hipError_t launch_pack_fill(dd_ctx *h, int which, hipStream_t st);
hipError_t launch_pack_unscaled(dd_ctx *h, hipStream_t st);
hipError_t launch_cast32(dd_ctx *h, hipStream_t st);
hipError_t launch_pack_slots(dd_ctx *h, int which, hipStream_t st);
// segmented slot layout of both sweeps: positions, wave-chunks, values
int build_seg_layout(dd_ctx *h, hipStream_t st);
hipError_t launch_seg_pack(dd_ctx *h, hipStream_t st);
// the wave-chunk table of a sweep of the slot layout
int build_wave_chunks(dd_ctx *h, int which, hipStream_t st);
hipError_t launch_export_factors(dd_ctx *h, double *f, hipStream_t st);
hipError_t launch_export_slots(dd_ctx *h, double *f, hipStream_t st);  // where launch_bilu0_slots factored
// out[k] = val[src[k]] for nblk blocks of bb values
hipError_t launch_gather_blocks(int64_t nblk, int bb, const int32_t *src, const double *val, double *out,
                                hipStream_t st);
// A's values in the reordered numbering (src: input block of each block) and
// the sliced ELL copy's values, from the caller's values
hipError_t launch_values(dd_ctx *h, const double *val, const int32_t *src, hipStream_t st);

hipError_t launch_apply(dd_ctx *h, const double *r, double *z, const int32_t *state,
                        hipStream_t st);
// nrhs applies of right-hand sides stored one after another (n*bs apart):
// one launch (grid.y = right-hand side) where the slot kernel runs, else one
// launch per right-hand side
hipError_t launch_apply_batch(dd_ctx *h, const double *r, double *z, int nrhs, hipStream_t st,
                              const int32_t *state = nullptr);
int apply_lds_bytes(const dd_ctx *h, int precision);
int spin_lds_bytes(const dd_ctx *h);
// 0 if the handle's precision and correction allow apply variant v, else the
// reason (for the ablation variants 4-8: FP64 only, no learned correction)
const char *variant_unsupported(const dd_ctx *h, int v);

// Krylov
hipError_t launch_spmv(dd_ctx *h, const double *x, double *y, hipStream_t st);
// memory and tables of the SpMV's sliced ELL copy of A (once per handle;
// launch_values writes the copy)
void build_spmv_layout(dd_ctx *h, hipStream_t st);
hipError_t launch_permute(int64_t n, int bs, const int32_t *map, const double *in, double *out,
                          hipStream_t st);
// vectors of n*bs in the Krylov workspace: ten for the recurrence, one to
// keep the initial guess while a learned solve may still fall back
constexpr int kKrylovVectors = 11;
// Device workspace of one solve: the Krylov vectors, the per-workgroup
// partial sums and the device scalars, plus a host copy of the scalars.
// Either the handle's own buffers (allocated on its first solve) or the
// library's fixed array (bicgstab_solve_noalloc).
struct KrylovWork {
    double *kv = nullptr;              // kKrylovVectors vectors of n*bs
    double *partials = nullptr;        // [8 * part_stride] per-workgroup partial sums
    int32_t part_stride = 0;
    KrylovScalars *ks = nullptr;       // device, three copies
    // host memory the device reports its iterations in (null: the host
    // synchronises every few iterations instead)
    unsigned long long *progress = nullptr;
    KrylovScalars *ks_host = nullptr;  // host (pinned for the handle's workspace)
    // false: create no HIP events (the solve is timed on the host, per-apply
    // profiling is off) and use no buffer outside this workspace (the fused
    // apply + SpMV launch, whose flags the handle allocates, is not used)
    bool handle_owned = true;
};
int bicgstab_run(dd_ctx *h, const KrylovWork &w, const double *b, double *x, double rtol, int32_t maxit,
                 hipStream_t st, dd_solve_info *info);
// the handle's Krylov workspace (allocated on the first call)
int krylov_workspace(dd_ctx *h, KrylovWork *w);
// the workspace in the library's fixed device array: no allocation;
// DD_EINVAL when the problem needs more than that array holds
int noalloc_workspace(dd_ctx *h, KrylovWork *w, KrylovScalars *host);
// bytes of the fixed array (per device)
constexpr int64_t kNoallocBytes = int64_t(128) << 20;

// global ILU0
int global_factor(dd_ctx *h, hipStream_t st);
hipError_t launch_global_apply(dd_ctx *h, const double *r, double *z, int nrhs, hipStream_t st);
hipError_t launch_gfactor_slots(dd_ctx *h, const std::vector<int32_t> &lp, hipStream_t st);
hipError_t launch_gapply_slots(dd_ctx *h, const double *r, double *z, int nrhs, hipStream_t st);
bool gapply_slots_fits(const dd_ctx *h, int halo);
hipError_t launch_diag_positions(dd_ctx *h, int32_t *diag, hipStream_t st);

// learned correction
int lic_setup(dd_ctx *h, hipStream_t st);
int lic_coeffs_from_params(dd_ctx *h, const float *params, bool keep_hidden, hipStream_t st);
// refresh the apply's rank-major copy of C after C changed
int lic_publish_coeffs(dd_ctx *h, hipStream_t st);
int lic_loss_grad_run(dd_ctx *h, const float *params, int Q, const double *R, const double *Zs, const double *den,
                      double *loss, float *grad, int accumulate, hipStream_t st);
int lic_targets_run(dd_ctx *h, int Q, const double *R, double *Zs, double *den, hipStream_t st);
hipError_t launch_adam(int np, float *P, const float *G, float *M, float *V, int t, float lr, float b1, float b2,
                       float eps, hipStream_t st);
// nrhs adjoint applies (right-hand sides n*3 apart) in one launch; the
// transposed streams must have been packed (lic_adjoint_streams)
hipError_t launch_apply_adjoint(dd_ctx *h, const double *g, double *a, int nrhs, hipStream_t st);
// pack the transposed factor streams of the adjoint apply (once per factorisation)
int lic_adjoint_streams(dd_ctx *h, hipStream_t st);
// the preconditioner bicgstab_solve uses (DD apply, or the global ILU0 apply)
// ev0/ev1 (optional): timing events around the apply; a slot-layout apply
// records them at its kernel's own start and end (hipExtLaunchKernel), any
// other path on the stream around its launches.
hipError_t launch_precond(dd_ctx *h, const double *r, double *z, const int32_t *state, hipStream_t st,
                          hipEvent_t ev0 = nullptr, hipEvent_t ev1 = nullptr);
constexpr int32_t kWaitFailed = -64;  // solve state word after a dependency wait hit its bound
// BiCGSTAB's apply and the SpMV behind it as one launch (mode 0: y = A z with
// the dot w.y; mode 1: the dots y.w and y.y), partials one per subdomain.
// Nonzero when the handle's shape or settings need the separate launches.
int fused_unsupported(const dd_ctx *h);
hipError_t launch_apply_spmv(dd_ctx *h, int mode, const double *r, double *z, double *y, const double *w,
                             double *part, int part_stride, uint32_t epoch, unsigned long long ticket0,
                             int32_t *state, hipStream_t st);
// dep[2k], dep[2k+1]: lowest and highest subdomain read by subdomain k's rows of A
hipError_t launch_dep_range(dd_ctx *h, hipStream_t st);
}  // namespace ddilu
