// Setup kernels: partition labels and permutation (Section 3, Algorithm 2),
// block reorder (Section 3.1, Algorithm 3), inter-subdomain drop (Section
// 3.2), per-subdomain level sets (Section 4.2.1), block ILU0 + ILDU0
// (Section 4.3, Algorithm 5) and the packing of the factors into the
// streaming layout of the apply.
#include <algorithm>

#include "blocks.h"
#include "internal.h"

namespace ddilu {

// ------------------------------------------------------------------ scan
constexpr int kScanT = 1024;
constexpr int kScanItems = 4;
constexpr int kScanTile = kScanT * kScanItems;

int64_t scan_tmp_elems(int64_t n) { return (n + kScanTile - 1) / kScanTile + 2; }

__global__ __launch_bounds__(kScanT) void k_scan_tiles(const int32_t *in, int64_t n, int32_t *sums) {
    __shared__ int sh[65];
    const int64_t t0 = (int64_t)blockIdx.x * kScanTile + (int64_t)threadIdx.x * kScanItems;
    int v = 0;
#pragma unroll
    for (int k = 0; k < kScanItems; ++k)
        if (t0 + k < n) v += in[t0 + k];
    int tot;
    block_excl_scan(v, sh, &tot);
    if (threadIdx.x == 0) sums[blockIdx.x] = tot;
}

__global__ __launch_bounds__(kScanT) void k_scan_sums(int32_t *sums, int64_t m) {
    __shared__ int sh[65];
    int carry = 0;
    for (int64_t base = 0; base < m; base += kScanT) {
        int64_t i = base + threadIdx.x;
        int v = i < m ? sums[i] : 0;
        int tot;
        int ex = block_excl_scan(v, sh, &tot);
        if (i < m) sums[i] = ex + carry;
        carry += tot;
    }
    if (threadIdx.x == 0) sums[m] = carry;
}

__global__ __launch_bounds__(kScanT) void k_scan_apply(const int32_t *in, int64_t n, const int32_t *sums,
                                                       int64_t m, int32_t *out) {
    __shared__ int sh[65];
    const int64_t t0 = (int64_t)blockIdx.x * kScanTile + (int64_t)threadIdx.x * kScanItems;
    int vals[kScanItems];
    int v = 0;
#pragma unroll
    for (int k = 0; k < kScanItems; ++k) {
        vals[k] = (t0 + k < n) ? in[t0 + k] : 0;
        v += vals[k];
    }
    int tot;
    int ex = block_excl_scan(v, sh, &tot) + sums[blockIdx.x];
#pragma unroll
    for (int k = 0; k < kScanItems; ++k) {
        if (t0 + k < n) out[t0 + k] = ex;
        ex += vals[k];
    }
    if (blockIdx.x == 0 && threadIdx.x == 0) out[n] = sums[m];
}

hipError_t exclusive_scan(const int32_t *in, int32_t *out, int64_t n, int32_t *tmp, hipStream_t st) {
    int64_t m = (n + kScanTile - 1) / kScanTile;
    if (m == 0) {
        return hipMemsetAsync(out, 0, sizeof(int32_t), st);
    }
    k_scan_tiles<<<(unsigned)m, kScanT, 0, st>>>(in, n, tmp);
    k_scan_sums<<<1, kScanT, 0, st>>>(tmp, m);
    k_scan_apply<<<(unsigned)m, kScanT, 0, st>>>(in, n, tmp, m, out);
    return hipGetLastError();
}

// ------------------------------------------------------------- partition
// Algorithm 2 label, and the renumbering of Section 3.1: rows grouped by
// label, stable in the old index.  Inside a box the stable order is the
// local lexicographic order, so the new index has the closed form
// part*S + li + sx*(lj + sy*lk).
__global__ void k_partition(int nx, int ny, int nz, int sx, int sy, int sz, int32_t *part_id,
                            int32_t *old2new, int32_t *new2old) {
    const int64_t n = (int64_t)nx * ny * nz;
    const int64_t g = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (g >= n) return;
    const int i = (int)(g % nx), j = (int)((g / nx) % ny), k = (int)(g / ((int64_t)nx * ny));
    const int bx = nx / sx, by = ny / sy;
    const int p = i / sx + bx * (j / sy + by * (k / sz));
    const int64_t S = (int64_t)sx * sy * sz;
    const int64_t loc = (i % sx) + (int64_t)sx * ((j % sy) + (int64_t)sy * (k % sz));
    const int64_t nw = p * S + loc;
    part_id[g] = p;
    old2new[g] = (int32_t)nw;
    new2old[nw] = (int32_t)g;
}

hipError_t launch_partition(dd_ctx *h, hipStream_t st) {
    const int T = 256;
    k_partition<<<(unsigned)((h->n + T - 1) / T), T, 0, st>>>(h->nx, h->ny, h->nz, h->sx, h->sy, h->sz,
                                                           h->part_id, h->old2new, h->new2old);
    return hipGetLastError();
}

// --------------------------------------------------------------- reorder
// Largest v of the workgroup, at most one atomic per workgroup (256 threads).
__device__ __forceinline__ void block_atomic_max(int v, int32_t *out) {
    __shared__ int wmax[4];
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) v = max(v, __shfl_xor(v, d));
    if ((threadIdx.x & 63) == 0) wmax[threadIdx.x >> 6] = v;
    __syncthreads();
    if (threadIdx.x == 0) {
        const int m = max(max(wmax[0], wmax[1]), max(wmax[2], wmax[3]));
        // a stale read only costs an atomic that does not change the maximum
        if (m > *const_cast<volatile int32_t *>(out)) atomicMax(out, m);
    }
}

// length of each reordered row; status[6] = the longest (one atomic per row
// serialises on the address: 375 us at 2M rows)
__global__ __launch_bounds__(256) void k_row_len(int64_t n, const int32_t *ptr, const int32_t *new2old, int32_t *len,
                                                int32_t *status) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    int32_t l = 0;
    if (i < n) {
        const int32_t o = new2old[i];
        l = ptr[o + 1] - ptr[o];
        len[i] = l;
        if (l < 0 || l > kMaxRowBlocks) atomicMax(&status[0], 1);
    }
    block_atomic_max(l, &status[6]);
}

// One thread per new row: map columns old->new and sort the row's
// (column, source block) pairs by column.  Rows of at most kRankRow blocks
// are sorted by counting (each pair's rank is the number of pairs before it,
// ties by position), all loads of the row in flight together and no pair
// moved twice; longer rows by insertion in place.
constexpr int kRankRow = 8;

__global__ void k_reorder_rows(int64_t n, const int32_t *__restrict__ ptr, const int32_t *__restrict__ col,
                               const int32_t *__restrict__ new2old, const int32_t *__restrict__ old2new,
                               const int32_t *__restrict__ aptr, int32_t *acol, int32_t *src) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const int32_t o = new2old[i];
    const int32_t b0 = ptr[o], len = ptr[o + 1] - b0;
    const int32_t d0 = aptr[i];
    if (len <= kRankRow) {
        int32_t c[kRankRow];
#pragma unroll
        for (int k = 0; k < kRankRow; ++k) c[k] = k < len ? old2new[col[b0 + k]] : 0x7fffffff;
#pragma unroll
        for (int k = 0; k < kRankRow; ++k) {
            if (k >= len) continue;
            int rank = 0;
#pragma unroll
            for (int j = 0; j < kRankRow; ++j) rank += (c[j] < c[k] || (c[j] == c[k] && j < k)) ? 1 : 0;
            acol[d0 + rank] = c[k];
            src[d0 + rank] = b0 + k;
        }
        return;
    }
    for (int k = 0; k < len; ++k) {
        int32_t c = old2new[col[b0 + k]];
        int32_t s = b0 + k;
        int m = k - 1;
        while (m >= 0 && acol[d0 + m] > c) {
            acol[d0 + m + 1] = acol[d0 + m];
            src[d0 + m + 1] = src[d0 + m];
            --m;
        }
        acol[d0 + m + 1] = c;
        src[d0 + m + 1] = s;
    }
}

__global__ void k_gather_blocks(int64_t nelem, int bb, const int32_t *src, const double *val, double *out) {
    const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= nelem) return;
    const int64_t q = e / bb;
    const int c = (int)(e - q * bb);
    out[e] = val[(int64_t)src[q] * bb + c];
}

// Input check before any kernel indexes through the caller's pattern: every
// row has 0..kMaxRowBlocks blocks inside [0, nnzb) (status[0] |= 1), every
// column is a block row (status[0] |= 2).
__global__ void k_check_rows(int64_t n, int64_t nnzb, const int32_t *ptr, const int32_t *col, int32_t *status) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const int32_t b0 = ptr[i], b1 = ptr[i + 1];
    if (b0 < 0 || b1 < b0 || b1 - b0 > kMaxRowBlocks || b1 > nnzb) {
        atomicOr(&status[0], 1);
        return;
    }
    for (int32_t q = b0; q < b1; ++q) {
        const int32_t c = col[q];
        if (c < 0 || c >= n) {
            atomicOr(&status[0], 2);
            return;
        }
    }
}

hipError_t launch_check_rows(int64_t n, int64_t nnzb, const int32_t *ptr, const int32_t *col, int32_t *status,
                             hipStream_t st) {
    const int T = 256;
    k_check_rows<<<(unsigned)((n + T - 1) / T), T, 0, st>>>(n, nnzb, ptr, col, status);
    return hipGetLastError();
}

hipError_t launch_row_len(dd_ctx *h, const int32_t *ptr, int32_t *len, hipStream_t st) {
    const int T = 256;
    k_row_len<<<(unsigned)((h->n + T - 1) / T), T, 0, st>>>(h->n, ptr, h->new2old, len, h->status);
    return hipGetLastError();
}

hipError_t launch_reorder_rows(dd_ctx *h, const int32_t *ptr, const int32_t *col, int32_t *src, hipStream_t st) {
    const int T = 256;
    k_reorder_rows<<<(unsigned)((h->n + T - 1) / T), T, 0, st>>>(h->n, ptr, col, h->new2old, h->old2new,
                                                              h->aptr, h->acol, src);
    return hipGetLastError();
}

// ------------------------------------------------------------------ drop
// Columns of a reordered row are sorted and a subdomain is the contiguous
// range [s*S, (s+1)*S), so the kept blocks of a row are one contiguous run.
__global__ void k_drop_count(int64_t n, int S, const int32_t *aptr, const int32_t *acol, int32_t *tbeg,
                             int32_t *tlen, int32_t *status) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const int64_t lo = (i / S) * (int64_t)S, hi = lo + S;
    int32_t b = aptr[i], e = aptr[i + 1];
    while (b < e && acol[b] < lo) ++b;
    int32_t f = b;
    bool diag = false;
    while (f < e && acol[f] < hi) {
        diag |= (acol[f] == i);
        ++f;
    }
    tbeg[i] = b;
    tlen[i] = f - b;
    if (!diag) atomicMin(&status[1], (int32_t)i);  // structurally missing pivot
}

__global__ void k_drop_rows(int64_t n, const int32_t *tbeg, const int32_t *tptr, const int32_t *acol,
                            int32_t *tcol, int32_t *tsrc, int32_t *tdiag) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const int32_t b = tbeg[i], d0 = tptr[i], len = tptr[i + 1] - d0;
    for (int k = 0; k < len; ++k) {
        const int32_t c = acol[b + k];
        tcol[d0 + k] = c;
        tsrc[d0 + k] = b + k;
        if (c == i) tdiag[i] = d0 + k;
    }
}

hipError_t launch_drop_count(dd_ctx *h, int32_t *tbeg, int32_t *tlen, hipStream_t st) {
    const int T = 256;
    k_drop_count<<<(unsigned)((h->n + T - 1) / T), T, 0, st>>>(h->n, h->S, h->aptr, h->acol, tbeg, tlen,
                                                            h->status);
    return hipGetLastError();
}

hipError_t launch_gather_blocks(int64_t nblk, int bb, const int32_t *src, const double *val, double *out,
                                hipStream_t st) {
    const int T = 256;
    const int64_t ne = nblk * bb;
    if (ne > 0) k_gather_blocks<<<(unsigned)((ne + T - 1) / T), T, 0, st>>>(ne, bb, src, val, out);
    return hipGetLastError();
}

hipError_t launch_drop_rows(dd_ctx *h, const int32_t *tbeg, int32_t *tsrc, hipStream_t st) {
    const int T = 256;
    k_drop_rows<<<(unsigned)((h->n + T - 1) / T), T, 0, st>>>(h->n, tbeg, h->tptr, h->acol, h->tcol, tsrc,
                                                           h->tdiag);
    return hipGetLastError();
}

// ------------------------------------------------------------------ BILU0
// Section 4.3, Algorithm 5 in block form, IKJ order, one workgroup per
// subdomain.  Rows are processed level by level (L levels): all rows a row
// depends on sit in earlier levels, so rows of one level run in parallel
// and each row performs exactly the sequential IKJ updates:
//   for each J < I in row I (ascending): L_IJ = U_IJ inv(U_JJ);
//     U_IK -= L_IJ U_JK for each K > J in row I that row J also holds.
// When a row is done its pivot inverse inv(U_II) is stored (it is the
// ILDU0 inv_D, and what later rows need).
template <int BS>
__global__ __launch_bounds__(256) void k_bilu0(int S, const int32_t *tptr, const int32_t *tcol,
                                               const int32_t *tdiag, double *lu, double *invd,
                                               const int32_t *nlev, const int32_t *off, const int32_t *lptr,
                                               const int32_t *rows, int32_t *status) {
    constexpr int BB = BS * BS;
    const int s = blockIdx.x;
    const int64_t base = (int64_t)s * S;
    const int nl = nlev[s];
    const int32_t o = off[s];
    for (int l = 0; l < nl; ++l) {
        const int32_t p0 = lptr[o + l], p1 = lptr[o + l + 1];
        for (int32_t p = p0 + threadIdx.x; p < p1; p += blockDim.x) {
            const int64_t gi = base + rows[base + p];
            const int32_t tb = tptr[gi], te = tptr[gi + 1];
            for (int32_t pj = tb; pj < te; ++pj) {
                const int32_t J = tcol[pj];
                if (J >= gi) break;
                double Lij[BB];
                blk_mul<BS>(lu + (int64_t)pj * BB, invd + (int64_t)J * BB, Lij);
#pragma unroll
                for (int e = 0; e < BB; ++e) lu[(int64_t)pj * BB + e] = Lij[e];
                const int32_t jb = tptr[J], je = tptr[J + 1];
                int32_t q = jb;
                for (int32_t pk = pj + 1; pk < te; ++pk) {
                    const int32_t K = tcol[pk];
                    while (q < je && tcol[q] < K) ++q;
                    if (q < je && tcol[q] == K) {
                        double t[BB];
                        blk_mul<BS>(Lij, lu + (int64_t)q * BB, t);
#pragma unroll
                        for (int e = 0; e < BB; ++e) lu[(int64_t)pk * BB + e] -= t[e];
                    }
                }
            }
            double inv[BB];
            const double *piv = lu + (int64_t)tdiag[gi] * BB;
            if (!blk_inverse<BS>(piv, inv)) {
                atomicMin(&status[2], (int32_t)gi);
#pragma unroll
                for (int e = 0; e < BB; ++e) inv[e] = (e % (BS + 1) == 0) ? 1.0 : 0.0;
            }
#pragma unroll
            for (int e = 0; e < BB; ++e) invd[gi * BB + e] = inv[e];
        }
        __syncthreads();
    }
}

hipError_t launch_bilu0(dd_ctx *h, hipStream_t st) {
    const Levels &L = h->lev[0];
    if (h->bs == 3)
        k_bilu0<3><<<h->nsub, 256, 0, st>>>(h->S, h->tptr, h->tcol, h->tdiag, h->lu, h->invd, L.nlev, L.off,
                                            L.ptr, L.rows, h->status);
    else
        k_bilu0<1><<<h->nsub, 256, 0, st>>>(h->S, h->tptr, h->tcol, h->tdiag, h->lu, h->invd, L.nlev, L.off,
                                            L.ptr, L.rows, h->status);
    return hipGetLastError();
}

// ------------------------------------------------------------------ pack
// Per position p of a sweep (subdomain s = p / S, row = rows[p]): the
// number of its factor blocks (lower: J < I; upper: K > I).
__global__ void k_pack_count(int64_t n, int S, int which, const int32_t *tptr, const int32_t *tcol,
                             const int32_t *rows, int32_t *cnt) {
    const int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= n) return;
    const int64_t gi = (p / S) * (int64_t)S + rows[p];
    int c = 0;
    for (int32_t q = tptr[gi]; q < tptr[gi + 1]; ++q) c += which == 0 ? (tcol[q] < gi) : (tcol[q] > gi);
    cnt[p] = c;
}

// which 0: L blocks; 1: Uhat = inv_D U blocks and inv_D; 2: the U blocks as
// factored (no scaling; val only, same order as for 1).
template <int BS>
__global__ void k_pack_fill(int64_t n, int S, int which, const int32_t *tptr, const int32_t *tcol,
                            const double *lu, const double *invd, const int32_t *rows, const int32_t *bptr,
                            uint16_t *prow, uint16_t *bcol, double *val, double *dval) {
    constexpr int BB = BS * BS;
    const int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= n) return;
    const int64_t base = (p / S) * (int64_t)S;
    const int64_t gi = base + rows[p];
    if (which != 2) prow[p] = (uint16_t)rows[p];
    int32_t b = bptr[p];
    const double *inv = invd + gi * BB;
    for (int32_t q = tptr[gi]; q < tptr[gi + 1]; ++q) {
        const int32_t c = tcol[q];
        if (which == 0 ? (c < gi) : (c > gi)) {
            if (which != 2) bcol[b] = (uint16_t)(c - base);
            if (which != 1) {
#pragma unroll
                for (int e = 0; e < BB; ++e) val[(int64_t)b * BB + e] = lu[(int64_t)q * BB + e];
            } else {
                double t[BB];
                blk_mul<BS>(inv, lu + (int64_t)q * BB, t);
#pragma unroll
                for (int e = 0; e < BB; ++e) val[(int64_t)b * BB + e] = t[e];
            }
            ++b;
        }
    }
    if (which == 1) {
#pragma unroll
        for (int e = 0; e < BB; ++e) dval[p * BB + e] = inv[e];
    }
}

hipError_t launch_pack_unscaled(dd_ctx *h, hipStream_t st) {
    const int T = 256;
    Sweep &w = h->sw[1];
    const unsigned g = (unsigned)((h->n + T - 1) / T);
    if (h->bs == 3)
        k_pack_fill<3><<<g, T, 0, st>>>(h->n, h->S, 2, h->tptr, h->tcol, h->lu, h->invd, h->lev[1].rows, w.bptr,
                                        nullptr, nullptr, w.uraw, nullptr);
    else
        k_pack_fill<1><<<g, T, 0, st>>>(h->n, h->S, 2, h->tptr, h->tcol, h->lu, h->invd, h->lev[1].rows, w.bptr,
                                        nullptr, nullptr, w.uraw, nullptr);
    return hipGetLastError();
}

hipError_t launch_pack_count(dd_ctx *h, int which, int32_t *cnt, hipStream_t st) {
    const int T = 256;
    k_pack_count<<<(unsigned)((h->n + T - 1) / T), T, 0, st>>>(h->n, h->S, which, h->tptr, h->tcol,
                                                            h->lev[which].rows, cnt);
    return hipGetLastError();
}

hipError_t launch_pack_fill(dd_ctx *h, int which, hipStream_t st) {
    const int T = 256;
    Sweep &w = h->sw[which];
    const unsigned g = (unsigned)((h->n + T - 1) / T);
    if (h->bs == 3)
        k_pack_fill<3><<<g, T, 0, st>>>(h->n, h->S, which, h->tptr, h->tcol, h->lu, h->invd, h->lev[which].rows,
                                        w.bptr, w.prow, w.bcol, w.val64, w.d64);
    else
        k_pack_fill<1><<<g, T, 0, st>>>(h->n, h->S, which, h->tptr, h->tcol, h->lu, h->invd, h->lev[which].rows,
                                        w.bptr, w.prow, w.bcol, w.val64, w.d64);
    return hipGetLastError();
}

// Slot layout of one sweep: position p owns MB block slots; its blocks fill
// the first nb slots in ascending column order, zero blocks the rest.  The
// position's 64-bit descriptor holds its local row in bits 0-15 and the
// local column of slot k in bits 16(k+1)..16(k+1)+15, 0xFFFF for an empty
// slot.
template <int BS>
__global__ void k_pack_slots(int64_t n, int S, int which, int MB, const int32_t *tptr, const int32_t *tcol,
                             const double *lu, const double *invd, const int32_t *rows, uint64_t *desc,
                             double *sval) {
    constexpr int BB = BS * BS;
    const int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= n) return;
    const int64_t base = (p / S) * (int64_t)S;
    const int32_t lr = rows[p];
    const int64_t gi = base + lr;
    const double *inv = invd + gi * BB;
    // lane-contiguous runs: row i of every slot block, then (upper sweep)
    // row i of inv_D, NV values per row i, PS = BS * NV per position
    const int NV = (MB + which) * BS;
    double *o = sval + p * BS * NV;
    uint64_t dsc = (uint64_t)(uint16_t)lr;
    int k = 0;
    for (int32_t q = tptr[gi]; q < tptr[gi + 1] && k < MB; ++q) {
        const int32_t c = tcol[q];
        if (which == 0 ? (c < gi) : (c > gi)) {
            dsc |= (uint64_t)(uint16_t)(c - base) << (16 * (k + 1));
            double t[BB];
            if (which == 0) {
#pragma unroll
                for (int e = 0; e < BB; ++e) t[e] = lu[(int64_t)q * BB + e];
            } else {
                blk_mul<BS>(inv, lu + (int64_t)q * BB, t);
            }
#pragma unroll
            for (int i = 0; i < BS; ++i)
#pragma unroll
                for (int j = 0; j < BS; ++j) o[i * NV + k * BS + j] = t[i * BS + j];
            ++k;
        }
    }
    for (int e = k; e < 3; ++e) dsc |= (uint64_t)0xffffu << (16 * (e + 1));
    for (; k < MB; ++k)
#pragma unroll
        for (int i = 0; i < BS; ++i)
#pragma unroll
            for (int j = 0; j < BS; ++j) o[i * NV + k * BS + j] = 0.0;
    if (which == 1)
#pragma unroll
        for (int i = 0; i < BS; ++i)
#pragma unroll
            for (int j = 0; j < BS; ++j) o[i * NV + MB * BS + j] = inv[i * BS + j];
    desc[p] = dsc;
}

hipError_t launch_pack_slots(dd_ctx *h, int which, hipStream_t st) {
    const int T = 256;
    Sweep &w = h->sw[which];
    const unsigned g = (unsigned)((h->n + T - 1) / T);
    if (h->bs == 3)
        k_pack_slots<3><<<g, T, 0, st>>>(h->n, h->S, which, h->slots, h->tptr, h->tcol, h->lu, h->invd,
                                         h->lev[which].rows, w.desc, w.sval64);
    else
        k_pack_slots<1><<<g, T, 0, st>>>(h->n, h->S, which, h->slots, h->tptr, h->tcol, h->lu, h->invd,
                                         h->lev[which].rows, w.desc, w.sval64);
    return hipGetLastError();
}

// Wave-chunks (see Sweep::wtab): one workgroup per subdomain walks its levels
// 256 at a time; a scan over the tile places each level's chunks.  A
// subdomain's chunks start at wbase: an upper bound of the chunks before it
// (a level of m positions has at most m/rpw + 1), so no count pass is needed.
__global__ __launch_bounds__(256) void k_wave_chunks(int S, int rpw, const int32_t *__restrict__ off,
                                                    const int32_t *__restrict__ lp, int2 *__restrict__ wtab,
                                                    int4 *__restrict__ winfo) {
    __shared__ int sh[65];
    const int s = blockIdx.x;
    const int32_t o = off[s];
    const int nl = off[s + 1] - o - 1;
    const int32_t wbase = (int32_t)((int64_t)s * S / rpw) + s + o;
    int chunks = 0;  // of the tiles before
    for (int t0 = 0; t0 < nl; t0 += blockDim.x) {
        const int l = t0 + threadIdx.x;
        int32_t q0 = 0, q1 = 0;
        if (l < nl) {
            q0 = lp[o + l];
            q1 = lp[o + l + 1];
        }
        const int m = (q1 - q0 + rpw - 1) / rpw;
        int tm;
        const int at = chunks + block_excl_scan(m, sh, &tm);
        for (int k = 0; k < m; ++k) {
            const int32_t p0 = q0 + k * rpw;
            wtab[wbase + at + k] = make_int2(p0, l << 8 | min(rpw, q1 - p0));
        }
        chunks += tm;
    }
    if (threadIdx.x == 0) winfo[s] = make_int4(wbase, chunks, nl, 0);
}

int build_wave_chunks(dd_ctx *h, int which, hipStream_t st) {
    Sweep &w = h->sw[which];
    const Levels &L = h->lev[which];
    const int rpw = kWave / h->bs;
    h->release(w.wtab);
    h->release(w.winfo);
    int rc = h->alloc(&w.wtab, w.snpos / rpw + h->nsub + L.ptr_len + 1);
    if (!rc) rc = h->alloc(&w.winfo, h->nsub);
    if (rc) return rc;
    k_wave_chunks<<<h->nsub, 256, 0, st>>>(h->S, rpw, L.off, L.ptr, w.wtab, w.winfo);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return h->fail(DD_EHIP, "wave chunks: %s", hipGetErrorString(e));
    return DD_OK;
}

// FP64 -> FP32 copies, round to nearest even.
__global__ void k_cast32(int64_t m, const double *in, float *out) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < m) out[i] = (float)in[i];
}

hipError_t launch_cast32(dd_ctx *h, hipStream_t st) {
    const int T = 256;
    const int bb = h->bs * h->bs;
    for (int w = 0; w < 2; ++w) {
        Sweep &s = h->sw[w];
        const int64_t m = s.val32 ? s.nblk * bb : 0;
        if (m) k_cast32<<<(unsigned)((m + T - 1) / T), T, 0, st>>>(m, s.val64, s.val32);
    }
    const int64_t m = h->n * bb;
    if (h->csr_ready && h->sw[1].d32) k_cast32<<<(unsigned)((m + T - 1) / T), T, 0, st>>>(m, h->sw[1].d64, h->sw[1].d32);
    if (h->slots || h->seg) {
        const int mb = h->seg ? h->seg : h->slots;
        for (int w = 0; w < 2; ++w) {
            const int64_t ms = h->sw[w].snpos * (mb + w) * bb;  // the upper stream carries inv_D
            if (ms) k_cast32<<<(unsigned)((ms + T - 1) / T), T, 0, st>>>(ms, h->sw[w].sval64, h->sw[w].sval32);
        }
    }
    return hipGetLastError();
}

// L\inv_D\Uhat in the dropped pattern (for inspection).
template <int BS>
__global__ void k_export(int64_t n, const int32_t *tptr, const int32_t *tcol, const double *lu,
                         const double *invd, double *f) {
    constexpr int BB = BS * BS;
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const double *inv = invd + i * BB;
    for (int32_t q = tptr[i]; q < tptr[i + 1]; ++q) {
        const int32_t c = tcol[q];
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

hipError_t launch_export_factors(dd_ctx *h, double *f, hipStream_t st) {
    if (h->direct) return launch_export_slots(h, f, st);
    const int T = 256;
    const unsigned g = (unsigned)((h->n + T - 1) / T);
    if (h->bs == 3)
        k_export<3><<<g, T, 0, st>>>(h->n, h->tptr, h->tcol, h->lu, h->invd, f);
    else
        k_export<1><<<g, T, 0, st>>>(h->n, h->tptr, h->tcol, h->lu, h->invd, f);
    return hipGetLastError();
}

}  // namespace ddilu
