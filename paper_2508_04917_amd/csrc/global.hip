// Global (undecomposed) ILU0 of the full reordered matrix: the preconditioner
// the decomposition approximates.  It serves as the regression target of the
// learned interface correction and as the reference for the iterations the
// decomposition costs.
//
// The level of a row is its longest dependency path in the whole matrix
// (Section 4.2.1).  The factorisation runs level by level, one launch each over
// the level's rows.  The apply runs, where the slot layout holds the factors,
// one launch per level of the subdomain graph, each subdomain's sweep with its
// vector and the rows it depends on in LDS (k_dd_apply_slots_global);
// otherwise one launch per level of the matrix, the vector in global memory.
//
// 48^3 3x3 blocks, 16^3 boxes, 16 probes: factorisation + targets 17.7 ms with
// every launch scanning all rows for its level (14.5 us each), a host
// synchronisation per relaxation step of the levels and the pattern's part
// done again on every call; 1.42 ms now, 2.2 ms on a handle's first call, which
// does the pattern's part; 142 factor launches are 0.81 ms of either, 14 sweep
// launches 0.38 ms.
#include <algorithm>

#include "blocks.h"
#include "internal.h"

namespace ddilu {

// Longest-path levels (blockIdx.y = 0: dependencies J < I, 1: J > I) of a
// tile of kTile consecutive rows, in place: the tile relaxes lev_I = max over
// its dependencies of lev_J + 1 in LDS until nothing in it changes, reading
// the levels of rows outside as they are.  Levels only grow, towards the
// longest path, so passes are repeated until one changes nothing; a chain
// costs a pass per tile it crosses instead of one per row (48^3 in 16^3
// boxes: 9 passes for 142 levels).
constexpr int kTile = 4096, kTileT = 1024;

__global__ __launch_bounds__(kTileT) void k_glev_tile(int64_t n, const int32_t *__restrict__ ptr,
                                                     const int32_t *__restrict__ col, int32_t *lev0, int32_t *lev1,
                                                     int32_t *changed) {
    __shared__ int32_t lv[kTile + 1];
    constexpr int R = kTile / kTileT;
    const int which = blockIdx.y, tid = threadIdx.x;
    int32_t *lev = which ? lev1 : lev0;
    const int64_t t0 = (int64_t)blockIdx.x * kTile;
    uint32_t d01[R], d23[R], more = 0;
    int32_t cur[R], old[R];
    if (tid == 0) lv[kTile] = -1;  // "no dependency"
    auto inside = [&](int64_t i, int32_t c, int32_t &at) {
        if (which ? c <= i : c >= i) return false;
        at = (int32_t)(c - t0);
        return true;
    };
#pragma unroll
    for (int k = 0; k < R; ++k) {
        const int64_t i = t0 + tid + k * kTileT;
        d01[k] = d23[k] = kTile | kTile << 16;
        cur[k] = old[k] = 0;
        if (i < n) {
            old[k] = lev[i];
            int32_t m = old[k];
            int cnt = 0;
            for (int32_t q = ptr[i]; q < ptr[i + 1]; ++q) {
                int32_t at;
                if (!inside(i, col[q], at)) continue;
                if (at < 0 || at >= kTile) {
                    m = max(m, lev[col[q]] + 1);
                } else {
                    if (cnt < 2)
                        d01[k] = cnt ? (d01[k] & 0xffffu) | (uint32_t)at << 16 : (uint32_t)at | (uint32_t)kTile << 16;
                    else if (cnt < 4)
                        d23[k] = cnt == 3 ? (d23[k] & 0xffffu) | (uint32_t)at << 16
                                          : (uint32_t)at | (uint32_t)kTile << 16;
                    else
                        more |= 1u << k;
                    ++cnt;
                }
            }
            cur[k] = m;
        }
        lv[tid + k * kTileT] = cur[k];
    }
    __syncthreads();
    for (;;) {
        asm volatile("" ::: "memory");
        bool moved = false;
#pragma unroll
        for (int k = 0; k < R; ++k) {
            int32_t m = max(max(lv[d01[k] & 0xffffu], lv[d01[k] >> 16]), max(lv[d23[k] & 0xffffu], lv[d23[k] >> 16])) + 1;
            if (more >> k & 1) {
                const int64_t i = t0 + tid + k * kTileT;
                for (int32_t q = ptr[i]; q < ptr[i + 1]; ++q) {
                    int32_t at;
                    if (inside(i, col[q], at) && at >= 0 && at < kTile) m = max(m, lv[at] + 1);
                }
            }
            if (m > cur[k]) {
                cur[k] = m;
                lv[tid + k * kTileT] = m;
                moved = true;
            }
        }
        if (!__syncthreads_or(moved)) break;
    }
    bool any = false;
#pragma unroll
    for (int k = 0; k < R; ++k) {
        const int64_t i = t0 + tid + k * kTileT;
        if (i < n && cur[k] != old[k]) {
            lev[i] = cur[k];
            any = true;
        }
    }
    if (any) *changed = 1;
}

__global__ __launch_bounds__(256) void k_gmax(int64_t n, const int32_t *__restrict__ lev0,
                                             const int32_t *__restrict__ lev1, int32_t *out) {
    __shared__ int32_t m;
    const int32_t *lev = blockIdx.y ? lev1 : lev0;
    if (threadIdx.x == 0) m = 0;
    __syncthreads();
    int32_t v = 0;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
        v = max(v, lev[i]);
    atomicMax(&m, v);
    __syncthreads();
    if (threadIdx.x == 0) atomicMax(&out[blockIdx.y], m);
}

// Rows of each level (their order inside a level is free: they are
// independent).  A workgroup counts its tile of rows per level in LDS and adds
// to (count) or takes its places from (place) each level's global counter
// once; more levels than the LDS table holds go to the counters row by row.
constexpr int kHist = 4096;

template <bool PLACE>
__global__ __launch_bounds__(kTileT) void k_glevel_rows(int64_t n, int nl, const int32_t *__restrict__ lev,
                                                       int32_t *counter, int32_t *__restrict__ list) {
    __shared__ int32_t cnt[kHist];
    const int64_t t0 = (int64_t)blockIdx.x * kTile, t1 = min(n, t0 + kTile);
    if (nl > kHist) {
        for (int64_t i = t0 + threadIdx.x; i < t1; i += blockDim.x) {
            const int32_t at = atomicAdd(&counter[lev[i]], 1);
            if (PLACE) list[at] = (int32_t)i;
        }
        return;
    }
    for (int l = threadIdx.x; l < nl; l += blockDim.x) cnt[l] = 0;
    __syncthreads();
    for (int64_t i = t0 + threadIdx.x; i < t1; i += blockDim.x) atomicAdd(&cnt[lev[i]], 1);
    __syncthreads();
    for (int l = threadIdx.x; l < nl; l += blockDim.x)
        if (cnt[l]) {
            const int32_t at = atomicAdd(&counter[l], cnt[l]);
            if (PLACE) cnt[l] = at;
        }
    if (!PLACE) return;
    __syncthreads();
    for (int64_t i = t0 + threadIdx.x; i < t1; i += blockDim.x) list[atomicAdd(&cnt[lev[i]], 1)] = (int32_t)i;
}

// Slot layout of the global factors: does every row have at most three blocks
// a sweep, no repeated block and updates of its pivot block only (bad[0]
// raised otherwise); and the number of each subdomain's halo rows (one
// workgroup per subdomain, blockIdx.y = sweep) or, with hrow given, the halo
// rows and the descriptors.
template <bool FILL>
__global__ __launch_bounds__(256) void k_ghalo(int S, const int32_t *__restrict__ ptr, const int32_t *__restrict__ col,
                                              const int32_t *__restrict__ diag, const int32_t *__restrict__ rows0,
                                              const int32_t *__restrict__ rows1, int32_t *cnt0, int32_t *cnt1,
                                              int32_t *__restrict__ hrow0, int32_t *__restrict__ hrow1,
                                              uint64_t *__restrict__ desc0, uint64_t *__restrict__ desc1,
                                              int32_t *bad) {
    __shared__ int sh[65];
    const int which = blockIdx.y, s = blockIdx.x;
    const int64_t base = (int64_t)s * S;
    const int32_t *rows = which ? rows1 : rows0;
    int32_t *cnt = which ? cnt1 : cnt0;  // FILL: first halo row of each subdomain
    int done = 0;
    for (int t0 = 0; t0 < S; t0 += blockDim.x) {
        const int p = t0 + threadIdx.x;
        int ext = 0;
        int32_t lo = 0, hi = 0, lr = 0;
        if (p < S) {
            lr = rows[base + p];
            const int64_t gi = base + lr;
            const int32_t d = diag[gi];
            lo = which ? d + 1 : ptr[gi];
            hi = which ? ptr[gi + 1] : d;
            for (int32_t q = lo; q < hi; ++q) {
                const int64_t c = col[q];
                ext += c < base || c >= base + S ? 1 : 0;
                if (!FILL && (c == gi || (q > lo && col[q - 1] == c))) bad[0] = 1;
            }
            if (!FILL && hi - lo > kMaxSlots) bad[0] = 1;
        }
        int tot;
        int at = done + block_excl_scan(ext, sh, &tot);
        if (FILL && p < S) {
            const int32_t h0 = cnt[s];
            uint64_t dsc = (uint64_t)(uint16_t)lr;
            for (int k = 0; k < kMaxSlots; ++k) {
                uint32_t f = 0xffff;
                if (lo + k < hi) {
                    const int64_t c = col[lo + k];
                    if (c < base || c >= base + S) {
                        (which ? hrow1 : hrow0)[h0 + at] = (int32_t)c;
                        f = (uint32_t)(S + at);
                        ++at;
                    } else {
                        f = (uint32_t)(c - base);
                    }
                }
                dsc |= (uint64_t)(f & 0xffff) << (16 * (k + 1));
            }
            (which ? desc1 : desc0)[base + p] = dsc;
        }
        done += tot;
    }
    if (!FILL && threadIdx.x == 0) {
        cnt[s] = done;
        atomicMax(&bad[1], done);
    }
}

// position of each row in the decomposed lower sweep
__global__ void k_ginv(int64_t n, int S, const int32_t *__restrict__ rows, int32_t *__restrict__ inv) {
    const int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (p < n) inv[p / S * S + rows[p]] = (int32_t)p;
}

// Factor records (see k_gfactor_slots) in level order; bad raised where a
// lower block's row shares another column with the row.
__global__ __launch_bounds__(256) void k_grecords(int64_t n, const int32_t *__restrict__ list,
                                                 const int32_t *__restrict__ ptr, const int32_t *__restrict__ col,
                                                 const int32_t *__restrict__ diag, const int32_t *__restrict__ linv,
                                                 const int32_t *__restrict__ uinv, int4 *__restrict__ rec,
                                                 int32_t *bad) {
    const int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= n) return;
    const int32_t i = list[p], tb = ptr[i], d = diag[i], te = ptr[i + 1];
    int32_t J[kMaxSlots], back[kMaxSlots];
    bool more = false;
    for (int k = 0; k < kMaxSlots; ++k) {
        J[k] = i;
        back[k] = -1;
        if (tb + k >= d) continue;
        J[k] = col[tb + k];
        for (int32_t r = diag[J[k]] + 1; r < ptr[J[k] + 1]; ++r) {
            const int32_t K = col[r];
            if (K == i)
                back[k] = r;
            else
                for (int32_t q = tb + k + 1; q < te; ++q) more |= col[q] == K;
        }
    }
    rec[3 * p] = make_int4(i, d, (d - tb) | (te - d - 1) << 8, linv[i]);
    rec[3 * p + 1] = make_int4(J[0], J[1], J[2], uinv[i]);
    rec[3 * p + 2] = make_int4(back[0], back[1], back[2], 0);
    if (more) *bad = 1;
}

__global__ void k_gdiag(int64_t n, const int32_t *__restrict__ ptr, const int32_t *__restrict__ col, int32_t *diag,
                        int32_t *status) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    int32_t d = -1;
    for (int32_t q = ptr[i]; q < ptr[i + 1]; ++q)
        if (col[q] == i) d = q;
    diag[i] = d;
    if (d < 0) atomicMin(&status[1], (int32_t)i);
}

// Block ILU0 (Algorithm 5, IKJ order) for the rows of one level.
template <int BS>
__global__ void k_gbilu0_level(int32_t p0, int32_t p1, const int32_t *__restrict__ list,
                               const int32_t *__restrict__ ptr, const int32_t *__restrict__ col,
                               const int32_t *__restrict__ diag, double *lu, double *invd, int32_t *status) {
    constexpr int BB = BS * BS;
    const int64_t p = p0 + (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= p1) return;
    const int64_t gi = list[p];
    const int32_t tb = ptr[gi], te = ptr[gi + 1];
    for (int32_t pj = tb; pj < te; ++pj) {
        const int32_t J = col[pj];
        if (J >= gi) break;
        double Lij[BB];
        blk_mul<BS>(lu + (int64_t)pj * BB, invd + (int64_t)J * BB, Lij);
#pragma unroll
        for (int e = 0; e < BB; ++e) lu[(int64_t)pj * BB + e] = Lij[e];
        const int32_t je = ptr[J + 1];
        int32_t q = ptr[J];
        for (int32_t pk = pj + 1; pk < te; ++pk) {
            const int32_t K = col[pk];
            while (q < je && col[q] < K) ++q;
            if (q < je && col[q] == K) {
                double t[BB];
                blk_mul<BS>(Lij, lu + (int64_t)q * BB, t);
#pragma unroll
                for (int e = 0; e < BB; ++e) lu[(int64_t)pk * BB + e] -= t[e];
            }
        }
    }
    double inv[BB];
    if (!blk_inverse<BS>(lu + (int64_t)diag[gi] * BB, inv)) {
        atomicMin(&status[2], (int32_t)gi);
#pragma unroll
        for (int e = 0; e < BB; ++e) inv[e] = (e % (BS + 1) == 0) ? 1.0 : 0.0;
    }
#pragma unroll
    for (int e = 0; e < BB; ++e) invd[gi * BB + e] = inv[e];
}

// ILDU0 form in the full pattern: L (lower), inv_D (diagonal), Uhat = inv_D U.
template <int BS>
__global__ void k_gildu0(int64_t n, const int32_t *__restrict__ ptr, const int32_t *__restrict__ col,
                         const double *__restrict__ lu, const double *__restrict__ invd, double *f) {
    constexpr int BB = BS * BS;
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const double *inv = invd + i * BB;
    for (int32_t q = ptr[i]; q < ptr[i + 1]; ++q) {
        const int32_t c = col[q];
        double t[BB];
        if (c < i) {
#pragma unroll
            for (int e = 0; e < BB; ++e) t[e] = lu[(int64_t)q * BB + e];
        } else if (c == i) {
#pragma unroll
            for (int e = 0; e < BB; ++e) t[e] = inv[e];
        } else {
            blk_mul<BS>(inv, lu + (int64_t)q * BB, t);
        }
#pragma unroll
        for (int e = 0; e < BB; ++e) f[(int64_t)q * BB + e] = t[e];
    }
}

// One level of the global forward (UPPER = false: y_I = r_I - sum_{J<I} L_IJ y_J,
// y kept in z) or backward sweep (z_I = inv_D_I y_I - sum_{K>I} Uhat_IK z_K).
// BS lanes of one wavefront per row; nrhs right-hand sides along grid y.
template <int BS, bool UPPER>
__global__ void k_gsweep_level(int64_t n, int32_t p0, int32_t p1, const int32_t *__restrict__ list,
                               const int32_t *__restrict__ ptr, const int32_t *__restrict__ col,
                               const int32_t *__restrict__ diag, const double *__restrict__ f,
                               const double *__restrict__ r, double *z) {
    constexpr int BB = BS * BS, RPW = kWave / BS;
    const int lane = threadIdx.x & 63;
    const int64_t gw = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) >> 6;
    const int64_t p = p0 + gw * RPW + lane / BS;
    const int c = lane % BS;
    const int64_t off = (int64_t)blockIdx.y * n * BS;
    if (lane / BS >= RPW || p >= p1) return;
    const int64_t i = list[p];
    const double *rr = r + off;
    double *zz = z + off;
    double acc;
    if constexpr (UPPER) {
        const double *dblk = f + (int64_t)diag[i] * BB + c * BS;
        acc = 0.0;
#pragma unroll
        for (int d = 0; d < BS; ++d) acc += dblk[d] * zz[i * BS + d];
    } else {
        acc = rr[i * BS + c];
    }
    for (int32_t q = ptr[i]; q < ptr[i + 1]; ++q) {
        const int64_t J = col[q];
        if (UPPER ? (J > i) : (J < i)) {
            const double *blk = f + (int64_t)q * BB + c * BS;
#pragma unroll
            for (int d = 0; d < BS; ++d) acc -= blk[d] * zz[J * BS + d];
        }
    }
    // the BS lanes of row i (one wavefront) have read z_i above
    __asm__ volatile("" ::: "memory");
    zz[i * BS + c] = acc;
}

hipError_t launch_diag_positions(dd_ctx *h, int32_t *diag, hipStream_t st) {
    const int T = 256;
    k_gdiag<<<(unsigned)((h->n + T - 1) / T), T, 0, st>>>(h->n, h->aptr, h->acol, diag, h->status);
    return hipGetLastError();
}

#define GCHK(x)                                                                             \
    do {                                                                                    \
        hipError_t e_ = (x);                                                                \
        if (e_ != hipSuccess) return h->fail(DD_EHIP, "%s: %s", #x, hipGetErrorString(e_)); \
    } while (0)
#define GRCHK(x)           \
    do {                   \
        int r_ = (x);      \
        if (r_) return r_; \
    } while (0)

// Level lists of the undecomposed matrix.
static int global_levels(dd_ctx *h, hipStream_t st) {
    const int T = 256;
    const unsigned g = (unsigned)((h->n + T - 1) / T), tiles = (unsigned)((h->n + kTile - 1) / kTile);
    for (int w = 0; w < 2; ++w) {
        if (!h->glev[w]) GRCHK(h->alloc(&h->glev[w], h->n));
        if (!h->glist[w]) GRCHK(h->alloc(&h->glist[w], h->n));
        GCHK(hipMemsetAsync(h->glev[w], 0, h->n * sizeof(int32_t), st));
    }
    int32_t *flag = h->status + 24;  // [0] changed, [1, 2] largest levels
    constexpr int kPasses = 4;       // between looks at the flag
    for (int64_t it = 0;; it += kPasses) {
        int32_t changed = 0;
        for (int k = 0; k < kPasses; ++k) {
            if (k == kPasses - 1) GCHK(hipMemsetAsync(flag, 0, sizeof(int32_t), st));
            k_glev_tile<<<dim3(tiles, 2), kTileT, 0, st>>>(h->n, h->aptr, h->acol, h->glev[0], h->glev[1], flag);
        }
        GCHK(hipMemcpyAsync(&changed, flag, sizeof(int32_t), hipMemcpyDeviceToHost, st));
        GCHK(hipStreamSynchronize(st));
        if (!changed) break;
        if (it > h->n + kPasses) return h->fail(DD_EINVAL, "global levels did not converge");
    }
    int32_t top[2] = {0, 0};
    GCHK(hipMemsetAsync(flag + 1, 0, sizeof(top), st));
    k_gmax<<<dim3(std::min(g, 1024u), 2), T, 0, st>>>(h->n, h->glev[0], h->glev[1], flag + 1);
    GCHK(hipMemcpyAsync(top, flag + 1, sizeof(top), hipMemcpyDeviceToHost, st));
    GCHK(hipStreamSynchronize(st));
    const int64_t most = std::max(top[0], top[1]) + 2;
    int32_t *cnt = nullptr, *cur = nullptr, *tmp = nullptr;
    int rc = h->alloc(&cnt, most);
    if (!rc) rc = h->alloc(&cur, most);
    if (!rc) rc = h->alloc(&tmp, scan_tmp_elems(most));
    for (int w = 0; w < 2 && !rc; ++w) {
        const int32_t nl = top[w] + 1;
        h->glp[w].assign(nl + 1, 0);
        hipError_t e = hipMemsetAsync(cnt, 0, nl * sizeof(int32_t), st);
        k_glevel_rows<false><<<tiles, kTileT, 0, st>>>(h->n, nl, h->glev[w], cnt, nullptr);
        if (e == hipSuccess) e = exclusive_scan(cnt, cur, nl, tmp, st);
        if (e == hipSuccess)
            e = hipMemcpyAsync(h->glp[w].data(), cur, (nl + 1) * sizeof(int32_t), hipMemcpyDeviceToHost, st);
        if (e == hipSuccess) e = hipStreamSynchronize(st);
        k_glevel_rows<true><<<tiles, kTileT, 0, st>>>(h->n, nl, h->glev[w], cur, h->glist[w]);
        if (e == hipSuccess) e = hipGetLastError();
        if (e == hipSuccess) e = hipStreamSynchronize(st);
        if (e != hipSuccess) rc = h->fail(DD_EHIP, "global levels: %s", hipGetErrorString(e));
    }
    h->release(cnt);
    h->release(cur);
    h->release(tmp);
    return rc;
}

// Halo rows, descriptors, records and the subdomain graph's levels, where the
// slot layout holds the global factors: the decomposed sweeps exist in slot
// form (their positions and chunk tables are shared), and a subdomain's
// vector fits the LDS together with its halo.
static int global_slots(dd_ctx *h, hipStream_t st) {
    h->gslots = 0;
    if (!h->patterned || !h->slots) return DD_OK;
    const int T = 256, bb = h->bs * h->bs;
    const unsigned g = (unsigned)((h->n + T - 1) / T);
    int32_t *bad = h->status + 24, got[2] = {0, 0}, *cnt[2] = {nullptr, nullptr};
    int rc = DD_OK;
    for (int w = 0; w < 2 && !rc; ++w) {
        rc = h->alloc(&cnt[w], h->nsub);
        if (!rc && !h->ghptr[w]) rc = h->alloc(&h->ghptr[w], h->nsub + 1);
    }
    auto bail = [&](int code) {
        for (int w = 0; w < 2; ++w) h->release(cnt[w]);
        return code;
    };
    if (rc) return bail(rc);
    const dim3 boxes(h->nsub, 2);
    hipError_t e = hipMemsetAsync(bad, 0, sizeof(got), st);
    k_ghalo<false><<<boxes, 256, 0, st>>>(h->S, h->aptr, h->acol, h->gdiag, h->lev[0].rows, h->lev[1].rows, cnt[0],
                                          cnt[1], nullptr, nullptr, nullptr, nullptr, bad);
    std::vector<int32_t> hp[2], hr[2];
    for (int w = 0; w < 2; ++w) {
        if (e == hipSuccess) e = exclusive_scan(cnt[w], h->ghptr[w], h->nsub, h->scan_tmp, st);
        hp[w].resize(h->nsub + 1);
        if (e == hipSuccess)
            e = hipMemcpyAsync(hp[w].data(), h->ghptr[w], hp[w].size() * sizeof(int32_t), hipMemcpyDeviceToHost, st);
    }
    if (e == hipSuccess) e = hipMemcpyAsync(got, bad, sizeof(got), hipMemcpyDeviceToHost, st);
    if (e == hipSuccess) e = hipStreamSynchronize(st);
    if (e != hipSuccess) return bail(h->fail(DD_EHIP, "global slots: %s", hipGetErrorString(e)));
    (void)bail(0);
    if (got[0] || !gapply_slots_fits(h, got[1])) return DD_OK;
    h->ghalo = got[1];
    int32_t *linv = nullptr;
    rc = h->alloc(&linv, h->n);
    for (int w = 0; w < 2 && !rc; ++w) {
        h->release(h->ghrow[w]);
        rc = h->alloc(&h->ghrow[w], hp[w].back());
        if (!rc && !h->gdesc[w]) rc = h->alloc(&h->gdesc[w], h->n);
        if (!rc && !h->gsval[w]) rc = h->alloc(&h->gsval[w], h->n * (kMaxSlots + w) * bb);
        if (!rc && !h->gbox[w]) rc = h->alloc(&h->gbox[w], h->nsub);
    }
    if (!rc && !h->grec) rc = h->alloc(&h->grec, 3 * h->n);
    if (!rc && !h->ginvd) rc = h->alloc(&h->ginvd, h->n * bb);
    if (rc) {
        h->release(linv);
        return rc;
    }
    k_ghalo<true><<<boxes, 256, 0, st>>>(h->S, h->aptr, h->acol, h->gdiag, h->lev[0].rows, h->lev[1].rows,
                                         h->ghptr[0], h->ghptr[1], h->ghrow[0], h->ghrow[1], h->gdesc[0], h->gdesc[1],
                                         bad);
    k_ginv<<<g, T, 0, st>>>(h->n, h->S, h->lev[0].rows, linv);
    k_grecords<<<g, T, 0, st>>>(h->n, h->glist[0], h->aptr, h->acol, h->gdiag, linv, h->uinv, h->grec, bad);
    e = hipGetLastError();
    for (int w = 0; w < 2; ++w) {
        hr[w].resize(hp[w].back());
        if (e == hipSuccess && !hr[w].empty())
            e = hipMemcpyAsync(hr[w].data(), h->ghrow[w], hr[w].size() * sizeof(int32_t), hipMemcpyDeviceToHost, st);
    }
    if (e == hipSuccess) e = hipMemcpyAsync(got, bad, sizeof(got), hipMemcpyDeviceToHost, st);
    if (e == hipSuccess) e = hipStreamSynchronize(st);
    h->release(linv);
    if (e != hipSuccess) return h->fail(DD_EHIP, "global slots: %s", hipGetErrorString(e));
    if (got[0]) return DD_OK;
    // levels of the subdomain graph: a subdomain only depends on lower
    // (upper sweep: higher) numbered ones, so one pass in that order does
    for (int w = 0; w < 2; ++w) {
        std::vector<int32_t> lev(h->nsub, 0), order(h->nsub);
        int32_t top = 0;
        for (int32_t k = 0; k < h->nsub; ++k) {
            const int32_t s = w ? h->nsub - 1 - k : k;
            for (int32_t q = hp[w][s]; q < hp[w][s + 1]; ++q) lev[s] = std::max(lev[s], lev[hr[w][q] / h->S] + 1);
            top = std::max(top, lev[s]);
        }
        std::vector<int32_t> &bp = h->gbp[w];
        bp.assign(top + 2, 0);
        for (int32_t s = 0; s < h->nsub; ++s) ++bp[lev[s] + 1];
        for (int32_t l = 0; l <= top; ++l) bp[l + 1] += bp[l];
        std::vector<int32_t> at(bp.begin(), bp.end() - 1);
        for (int32_t s = 0; s < h->nsub; ++s) order[at[lev[s]]++] = s;
        GCHK(hipMemcpyAsync(h->gbox[w], order.data(), h->nsub * sizeof(int32_t), hipMemcpyHostToDevice, st));
        GCHK(hipStreamSynchronize(st));
    }
    h->gslots = 1;
    return DD_OK;
}

int global_factor(dd_ctx *h, hipStream_t st) {
    const int bb = h->bs * h->bs, T = 256;
    const unsigned g = (unsigned)((h->n + T - 1) / T);
    ReclaimAtExit at_exit{h};
    int32_t init_status[8] = {0, 0x7fffffff, 0x7fffffff, 0, 0, 0, 0, 0}, status[8];
    GCHK(hipMemcpyAsync(h->status, init_status, sizeof(init_status), hipMemcpyHostToDevice, st));
    // the pattern's part, once per handle (again when the decomposed sweeps,
    // whose positions the slot layout shares, have been built since)
    if (!h->gpattern || (!h->gslots && h->gpattern == 1 && h->patterned && h->slots)) {
        if (!h->gpattern) {
            if (!h->gdiag) GRCHK(h->alloc(&h->gdiag, h->n));
            k_gdiag<<<g, T, 0, st>>>(h->n, h->aptr, h->acol, h->gdiag, h->status);
            GRCHK(global_levels(h, st));
        }
        GCHK(hipMemcpyAsync(status, h->status, sizeof(status), hipMemcpyDeviceToHost, st));
        GCHK(hipStreamSynchronize(st));
        if (status[1] != 0x7fffffff) return h->fail(DD_EZEROPIVOT, "block row %d has no diagonal block", status[1]);
        h->gpattern = h->patterned ? 2 : 1;
        GRCHK(global_slots(h, st));
    }
    h->gfactored = 0;
    if (h->gslots) {
        GCHK(launch_gfactor_slots(h, h->glp[0], st));
    } else {
        if (!h->glu) GRCHK(h->alloc(&h->glu, h->nnzb * bb));
        if (!h->ginvd) GRCHK(h->alloc(&h->ginvd, h->n * bb));
        if (!h->gf) GRCHK(h->alloc(&h->gf, h->nnzb * bb));
        GCHK(hipMemcpyAsync(h->glu, h->aval, h->nnzb * bb * sizeof(double), hipMemcpyDeviceToDevice, st));
        const std::vector<int32_t> &lp = h->glp[0];
        for (size_t l = 0; l + 1 < lp.size(); ++l) {
            const unsigned gl = (unsigned)((lp[l + 1] - lp[l] + 63) / 64);
            if (h->bs == 3)
                k_gbilu0_level<3><<<gl, 64, 0, st>>>(lp[l], lp[l + 1], h->glist[0], h->aptr, h->acol, h->gdiag,
                                                     h->glu, h->ginvd, h->status);
            else
                k_gbilu0_level<1><<<gl, 64, 0, st>>>(lp[l], lp[l + 1], h->glist[0], h->aptr, h->acol, h->gdiag,
                                                     h->glu, h->ginvd, h->status);
        }
        if (h->bs == 3)
            k_gildu0<3><<<g, T, 0, st>>>(h->n, h->aptr, h->acol, h->glu, h->ginvd, h->gf);
        else
            k_gildu0<1><<<g, T, 0, st>>>(h->n, h->aptr, h->acol, h->glu, h->ginvd, h->gf);
    }
    GCHK(hipGetLastError());
    GCHK(hipMemcpyAsync(status, h->status, sizeof(status), hipMemcpyDeviceToHost, st));
    GCHK(hipStreamSynchronize(st));
    if (status[2] != 0x7fffffff)
        return h->fail(DD_EZEROPIVOT, "global ILU0: singular pivot at reordered block row %d", status[2]);
    h->gfactored = 1;
    return DD_OK;
}

hipError_t launch_global_apply(dd_ctx *h, const double *r, double *z, int nrhs, hipStream_t st) {
    if (h->gslots) return launch_gapply_slots(h, r, z, nrhs, st);
    const int T = 256;
    const int rpb = (kWave / h->bs) * (T / kWave);
    for (int w = 0; w < 2; ++w) {
        const std::vector<int32_t> &lp = h->glp[w];
        for (size_t l = 0; l + 1 < lp.size(); ++l) {
            const dim3 grid((unsigned)((lp[l + 1] - lp[l] + rpb - 1) / rpb), (unsigned)nrhs);
            auto go = [&](auto kern) {
                kern<<<grid, T, 0, st>>>(h->n, lp[l], lp[l + 1], h->glist[w], h->aptr, h->acol, h->gdiag, h->gf, r, z);
            };
            if (h->bs == 3) {
                if (w) go(k_gsweep_level<3, true>); else go(k_gsweep_level<3, false>);
            } else {
                if (w) go(k_gsweep_level<1, true>); else go(k_gsweep_level<1, false>);
            }
        }
    }
    return hipGetLastError();
}

}  // namespace ddilu
