// Level sets (Section 4.2.1, 4.2.2) and the numeric factorisation of the slot
// layout (Section 4.3, Algorithm 5): block ILU0, the ILDU0 scaling and the
// packing of both sweeps' streams in one pass over the matrix.
#include <algorithm>

#include "blocks.h"
#include "internal.h"

namespace ddilu {

// Positions of row gi's lower (which = 0: columns < gi) or upper blocks in
// the dropped pattern (columns sorted; a repeated diagonal block belongs to
// neither).
__device__ __forceinline__ void dep_range(int which, int64_t gi, const int32_t *__restrict__ tptr,
                                          const int32_t *__restrict__ tcol, const int32_t *__restrict__ tdiag,
                                          int32_t &lo, int32_t &hi) {
    lo = which ? tdiag[gi] + 1 : tptr[gi];
    hi = which ? tptr[gi + 1] : tdiag[gi];
    if (which)
        while (lo < hi && tcol[lo] <= gi) ++lo;
    else
        while (lo < hi && tcol[hi - 1] >= gi) --hi;
}

// ---------------------------------------------------------------- levels
// Algorithm 6 semantics: inside one subdomain (one workgroup, grid y = sweep),
// rows without a dependency get level 0, every other row 1 + the largest
// level among its dependencies: the columns J < I (lower) or K > I (upper).
// Latency-bound: as many rounds as levels.  Each thread keeps its rows'
// first four dependencies in registers (R rows of 1,024 lanes; R = 0: read
// from memory each round), so a round is LDS reads of levels only, and a
// wavefront repeats its rows until none of them advances before it meets the
// others at a barrier (a chain inside 64 consecutive rows takes no barrier).
// A level once written is final, so it does not matter in which round
// another wavefront's write is seen.  2,097,152 rows in 512 boxes of 16^3,
// both sweeps: 2,470 us with the columns read again in every round -> 314 us.
constexpr uint16_t kNoLevel = 0xffff;
constexpr int kLevT = 1024;

template <int R>
__global__ __launch_bounds__(kLevT) void k_level_sets(int S, const int32_t *__restrict__ tptr,
                                                     const int32_t *__restrict__ tcol,
                                                     const int32_t *__restrict__ tdiag, int32_t *__restrict__ lev0,
                                                     int32_t *__restrict__ lev1, int32_t *__restrict__ nlev0,
                                                     int32_t *__restrict__ nlev1, int32_t *__restrict__ stats) {
    extern __shared__ uint16_t lev[];
    __shared__ int top, widest, blocks;
    constexpr int RR = R > 0 ? R : 1;
    const int which = blockIdx.y, s = blockIdx.x, tid = threadIdx.x, nt = blockDim.x;
    const int64_t base = (int64_t)s * S;
    auto range = [&](int i, int32_t &lo, int32_t &hi) { dep_range(which, base + i, tptr, tcol, tdiag, lo, hi); };
    uint32_t d01[RR], d23[RR];       // a row's first four dependencies (repeated when it has fewer)
    uint32_t pend = 0, more = 0;     // rows without a level; rows with more than four dependencies
    int most = 0, sum = 0;
    if (tid == 0) {
        top = 0;
        widest = 0;
        blocks = 0;
    }
    auto first = [&](int i, int k) {
        int32_t lo, hi;
        range(i, lo, hi);
        most = max(most, hi - lo);
        sum += hi - lo;
        lev[i] = hi > lo ? kNoLevel : 0;
        if (R > 0 && hi > lo) {
            auto c = [&](int j) { return (uint32_t)(tcol[min(lo + j, hi - 1)] - base) & 0xffffu; };
            d01[k] = c(0) | c(1) << 16;
            d23[k] = c(2) | c(3) << 16;
            pend |= 1u << k;
            if (hi - lo > 4) more |= 1u << k;
        }
    };
    if constexpr (R > 0) {
#pragma unroll
        for (int k = 0; k < RR; ++k) {
            d01[k] = d23[k] = 0;
            if (tid + k * nt < S) first(tid + k * nt, k);
            if (k % 4 == 3) __builtin_amdgcn_sched_barrier(0);  // bounds the loads' registers
        }
    } else {
        for (int i = tid; i < S; i += nt) first(i, 0);
    }
    __syncthreads();
    // largest level of row i's dependencies, kNoLevel if one has none yet
    auto rest = [&](int i) {
        int32_t lo, hi;
        range(i, lo, hi);
        int m = 0;
        for (int32_t q = lo; q < hi && m != kNoLevel; ++q) m = max(m, (int)lev[tcol[q] - base]);
        return m;
    };
    for (;;) {
        bool left;
        for (;;) {
            asm volatile("" ::: "memory");  // levels written since are read again
            bool moved = false;
            left = false;
            if constexpr (R > 0) {
                constexpr int G = RR < 4 ? RR : 4;  // rows whose reads are in flight together
                uint32_t longer = 0;  // rows whose first four dependencies have levels, and which have more
#pragma unroll
                for (int k0 = 0; k0 < RR; k0 += G) {
                    int m[G];
#pragma unroll
                    for (int g = 0; g < G; ++g) {
                        const uint32_t a = d01[k0 + g], b = d23[k0 + g];
                        m[g] = max(max((int)lev[a & 0xffff], (int)lev[a >> 16]),
                                   max((int)lev[b & 0xffff], (int)lev[b >> 16]));
                    }
                    const uint32_t before = pend;
#pragma unroll
                    for (int g = 0; g < G; ++g) {
                        const int k = k0 + g;
                        if ((pend >> k & 1) && m[g] != kNoLevel) {
                            if (more >> k & 1) {
                                longer |= 1u << k;
                            } else {
                                lev[tid + k * nt] = (uint16_t)(m[g] + 1);
                                pend &= ~(1u << k);
                            }
                        }
                    }
                    moved |= pend != before;
                    __builtin_amdgcn_sched_barrier(0);
                }
                while (longer) {
                    const int k = __ffs(longer) - 1;
                    longer &= longer - 1;
                    const int v = rest(tid + k * nt);
                    if (v != kNoLevel) {
                        lev[tid + k * nt] = (uint16_t)(v + 1);
                        pend &= ~(1u << k);
                        moved = true;
                    }
                }
                left = pend != 0;
            } else {
                for (int i = tid; i < S; i += nt)
                    if (lev[i] == kNoLevel) {
                        const int m = rest(i);
                        if (m != kNoLevel) {
                            lev[i] = (uint16_t)(m + 1);
                            moved = true;
                        } else {
                            left = true;
                        }
                    }
            }
            if (!__any(moved)) break;
        }
        if (!__syncthreads_or(left)) break;
    }
    int m = 0;
    int32_t *out = which ? lev1 : lev0;
    for (int i = tid; i < S; i += nt) {
        const int l = lev[i];
        m = max(m, l);
        out[base + i] = l;
    }
    atomicMax(&top, m);
    atomicMax(&widest, most);
    atomicAdd(&blocks, sum);
    __syncthreads();
    if (tid == 0) {
        (which ? nlev1 : nlev0)[s] = top + 1;
        atomicMax(&stats[which], widest);
        atomicMax(&stats[2 + which], top + 1);
        atomicAdd(&stats[6 + which], blocks);
    }
}

__global__ void k_plus_one(int64_t m, const int32_t *in, int32_t *out) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < m) out[i] = in[i] + 1;
}

// Explicit DAG (Section 4.2.2): per subdomain and sweep, level offsets and the
// rows of each level in ascending local order: a stable counting sort by
// level.  Each wavefront owns a contiguous run of rows; it counts them per
// level, the counts are scanned level by level and wavefront by wavefront,
// and it places its rows 64 at a time, equal levels ranked by lane.  linv,
// uinv: position of each row.  2,097,152 rows, both sweeps: 790 us
// with one thread per subdomain -> 68 us.
constexpr int kSortLevels = 1024;  // one level per thread in the scan

__global__ __launch_bounds__(kLevT) void k_level_sort(int S, const int32_t *__restrict__ lev0,
                                                     const int32_t *__restrict__ lev1,
                                                     const int32_t *__restrict__ nlev0,
                                                     const int32_t *__restrict__ nlev1,
                                                     const int32_t *__restrict__ off0,
                                                     const int32_t *__restrict__ off1, int32_t *__restrict__ ptr0,
                                                     int32_t *__restrict__ ptr1, int32_t *__restrict__ rows0,
                                                     int32_t *__restrict__ rows1, int32_t *__restrict__ linv,
                                                     int32_t *__restrict__ uinv,
                                                     int32_t *__restrict__ stats) {
    extern __shared__ int32_t cnt[];  // [wavefronts][levels]
    __shared__ int sh[65];
    __shared__ int widest;
    const int which = blockIdx.y, s = blockIdx.x, tid = threadIdx.x, nt = blockDim.x;
    const int lane = tid & (kWave - 1), w = tid / kWave, nw = nt / kWave;
    const int64_t base = (int64_t)s * S;
    const int32_t *lev = (which ? lev1 : lev0) + base;
    const int nl = (which ? nlev1 : nlev0)[s];
    int32_t *lptr = (which ? ptr1 : ptr0) + (which ? off1 : off0)[s];
    int32_t *rows = (which ? rows1 : rows0) + base;
    for (int i = tid; i < nw * nl; i += nt) cnt[i] = 0;
    if (tid == 0) widest = 0;
    __syncthreads();
    const int run = (S + nt - 1) / nt * kWave, r0 = w * run, r1 = min(S, r0 + run);
    for (int i = r0 + lane; i < r1; i += kWave) atomicAdd(&cnt[w * nl + lev[i]], 1);
    __syncthreads();
    int tot = 0;
    if (tid < nl)
        for (int k = 0; k < nw; ++k) {
            const int c = cnt[k * nl + tid];
            cnt[k * nl + tid] = tot;
            tot += c;
        }
    int all;
    const int start = block_excl_scan(tot, sh, &all);
    if (tid < nl) {
        lptr[tid] = start;
        for (int k = 0; k < nw; ++k) cnt[k * nl + tid] += start;
        atomicMax(&widest, tot);
    }
    if (tid == 0) lptr[nl] = S;
    __syncthreads();
    if (tid == 0) atomicMax(&stats[4], widest);
    volatile int32_t *at = cnt + w * nl;  // only this wavefront's from here on
    for (int i0 = r0; i0 < r1; i0 += kWave) {
        const int i = i0 + lane;
        const int l = i < r1 ? lev[i] : -1;
        unsigned long long todo = __ballot(l >= 0);
        while (todo) {
            const int lead = __ffsll(todo) - 1;
            const int ll = __shfl(l, lead);
            const unsigned long long same = __ballot(l == ll);
            const int p0 = at[ll];
            if (l == ll) {
                const int p = p0 + __popcll(same & ((1ull << lane) - 1));
                rows[p] = i;
                (which ? uinv : linv)[base + i] = (int32_t)(base + p);
            }
            if (lane == lead) at[ll] = p0 + __popcll(same);
            todo &= ~same;
        }
    }
}

// The same sort by one thread per subdomain, for subdomains of more levels
// than k_level_sort scans.
__global__ void k_level_lists(int S, int which, const int32_t *lev_g, const int32_t *nlev, const int32_t *off,
                              int32_t *lptr, int32_t *rows, int32_t *inv, int32_t *stats) {
    extern __shared__ int32_t sm_ll[];
    int32_t *cnt = sm_ll;                                       // nl + 1
    uint16_t *lv = reinterpret_cast<uint16_t *>(sm_ll + S + 1);  // S
    const int s = blockIdx.x;
    const int64_t base = (int64_t)s * S;
    const int nl = nlev[s];
    for (int i = threadIdx.x; i < S; i += blockDim.x) lv[i] = (uint16_t)lev_g[base + i];
    for (int l = threadIdx.x; l <= nl; l += blockDim.x) cnt[l] = 0;
    __syncthreads();
    if (threadIdx.x == 0) {
        int widest = 0;
        for (int i = 0; i < S; ++i) cnt[lv[i] + 1]++;
        for (int l = 0; l < nl; ++l) {
            widest = max(widest, cnt[l + 1]);
            cnt[l + 1] += cnt[l];
        }
        const int32_t o = off[s];
        for (int l = 0; l <= nl; ++l) lptr[o + l] = cnt[l];
        for (int i = 0; i < S; ++i) {
            const int p = cnt[lv[i]]++;
            rows[base + p] = i;
            inv[base + i] = (int32_t)(base + p);
        }
        atomicMax(&stats[4], widest);
    }
}

template <typename K>
static hipError_t full_lds(K kern) {
    return hipFuncSetAttribute(reinterpret_cast<const void *>(kern), hipFuncAttributeMaxDynamicSharedMemorySize,
                               163840 - 1024);
}

hipError_t launch_level_sets(dd_ctx *h, int32_t *stats, hipStream_t st) {
    Levels &L = h->lev[0], &U = h->lev[1];
    // four rows a thread where 1,024 threads allow it
    const int nt = std::min(kLevT, (h->S + 4 * kWave - 1) / (4 * kWave) * kWave);
    const int r = (h->S + nt - 1) / nt;
    auto go = [&](auto kern) -> hipError_t {
        hipError_t e = full_lds(kern);
        if (e != hipSuccess) return e;
        kern<<<dim3(h->nsub, 2), nt, (size_t)h->S * 2, st>>>(h->S, h->tptr, h->tcol, h->tdiag, L.lev, U.lev, L.nlev,
                                                             U.nlev, stats);
        return hipGetLastError();
    };
    if (r <= 4) return go(k_level_sets<4>);
    if (r <= 8) return go(k_level_sets<8>);
    if (r <= 20) return go(k_level_sets<20>);
    return go(k_level_sets<0>);
}

hipError_t launch_plus_one(int64_t m, const int32_t *in, int32_t *out, hipStream_t st) {
    const int T = 256;
    k_plus_one<<<(unsigned)((m + T - 1) / T), T, 0, st>>>(m, in, out);
    return hipGetLastError();
}

hipError_t launch_level_lists(dd_ctx *h, int32_t *stats, hipStream_t st) {
    Levels &L = h->lev[0], &U = h->lev[1];
    const int nl = std::max(L.max_levels, U.max_levels);
    if (nl <= kSortLevels) {
        // as many threads as levels need, at most as many wavefronts as 64 KB of counts hold
        int nt = std::min(kLevT, (h->S + kWave - 1) / kWave * kWave);
        nt = std::max(nt, (nl + kWave - 1) / kWave * kWave);
        hipError_t e = full_lds(k_level_sort);
        if (e != hipSuccess) return e;
        k_level_sort<<<dim3(h->nsub, 2), nt, (size_t)(nt / kWave) * nl * sizeof(int32_t), st>>>(
            h->S, L.lev, U.lev, L.nlev, U.nlev, L.off, U.off, L.ptr, U.ptr, L.rows, U.rows, h->linv, h->uinv, stats);
        return hipGetLastError();
    }
    const size_t lds = (size_t)(h->S + 1) * 4 + (size_t)h->S * 2;
    hipError_t e = full_lds(k_level_lists);
    if (e != hipSuccess) return e;
    for (int w = 0; w < 2; ++w)
        k_level_lists<<<h->nsub, 64, lds, st>>>(h->S, w, h->lev[w].lev, h->lev[w].nlev, h->lev[w].off, h->lev[w].ptr,
                                                h->lev[w].rows, w ? h->uinv : h->linv, stats);
    return hipGetLastError();
}

// ------------------------------------------------- factor into the slot layout
// Descriptors of one sweep's slots (see k_pack_slots): local row and the
// local columns of the row's lower or upper blocks in ascending order.
__global__ __launch_bounds__(256) void k_slot_desc(int64_t n, int S, const int32_t *__restrict__ tptr,
                                                  const int32_t *__restrict__ tcol,
                                                  const int32_t *__restrict__ tdiag,
                                                  const int32_t *__restrict__ rows0,
                                                  const int32_t *__restrict__ rows1, uint64_t *__restrict__ desc0,
                                                  uint64_t *__restrict__ desc1) {
    const int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= n) return;
    const int which = blockIdx.y;
    const int64_t base = (p / S) * (int64_t)S;
    const int32_t lr = (which ? rows1 : rows0)[p];
    const int64_t gi = base + lr;
    int32_t lo, hi;
    dep_range(which, gi, tptr, tcol, tdiag, lo, hi);
    uint64_t d = (uint64_t)(uint16_t)lr;
#pragma unroll
    for (int k = 0; k < kMaxSlots; ++k)
        d |= (uint64_t)(uint16_t)(lo + k < hi ? tcol[lo + k] - (int32_t)base : 0xffff) << (16 * (k + 1));
    (which ? desc1 : desc0)[p] = d;
}

// What the numeric factorisation needs of a row besides its lower descriptor,
// in lower-sweep order: {first block of the row in A's array, in the dropped
// pattern, upper-sweep position, lower blocks | upper blocks << 8} and, per
// lower block L_IJ, the position in A's array of A_JI (-1 where row J has no
// block in column I).  When a lower block's row J shares another column
// K > J with row I, ILU0 updates more than the pivot block: stats[0] is raised
// and the general kernel (k_bilu0) factors the matrix.
__global__ __launch_bounds__(256) void k_factor_records(int64_t n, int S, const int32_t *__restrict__ tptr,
                                                       const int32_t *__restrict__ tcol,
                                                       const int32_t *__restrict__ tdiag,
                                                       const int32_t *__restrict__ tsrc,
                                                       const int32_t *__restrict__ rows0,
                                                       const int32_t *__restrict__ linv,
                                                       const int32_t *__restrict__ uinv, int4 *__restrict__ rec,
                                                       int32_t *__restrict__ stats) {
    __shared__ int far;
    // threads past the end repeat the last position
    const int64_t p = min((int64_t)blockIdx.x * blockDim.x + threadIdx.x, n - 1);
    if (threadIdx.x == 0) far = 0;
    __syncthreads();
    const int64_t base = (p / S) * (int64_t)S, gi = base + rows0[p];
    const int32_t tb = tptr[gi], td = tdiag[gi], te = tptr[gi + 1];
    constexpr int ML = 2 * kMaxSlots + 1;  // blocks of a row of the slot layout
    int32_t c[ML], back[kMaxSlots];
    bool more = te - tb > ML;
#pragma unroll
    for (int j = 0; j < ML; ++j) c[j] = tcol[min(tb + j, te - 1)];
#pragma unroll
    for (int j = 1; j < ML; ++j) more |= tb + j < te && c[j] == c[j - 1];  // repeated blocks
    int32_t jd[kMaxSlots], je[kMaxSlots], jp[kMaxSlots], back_by = 0;
#pragma unroll
    for (int k = 0; k < kMaxSlots; ++k) {
        const int32_t J = tb + k < td ? c[k] : (int32_t)gi;
        jd[k] = tdiag[J];
        je[k] = tptr[J + 1];
        jp[k] = linv[J];
    }
#pragma unroll
    for (int k = 0; k < kMaxSlots; ++k) {
        back[k] = -1;
        back_by = max(back_by, (int32_t)p - jp[k]);
        int32_t at = -1;
#pragma unroll
        for (int u = 1; u <= kMaxSlots; ++u) {
            const int32_t K = tcol[min(jd[k] + u, je[k] - 1)];
            const bool in = tb + k < td && jd[k] + u < je[k];
            if (in && K == gi) at = jd[k] + u;
#pragma unroll
            for (int q = k + 1; q < ML; ++q) more |= in && K != gi && tb + q < te && c[q] == K;
        }
        if (at >= 0) back[k] = tsrc[at];
    }
    auto local = [&](int32_t q) { return (uint32_t)(q - base) & 0xffffu; };
    rec[2 * p] = make_int4(tsrc[tb], tb, uinv[gi],
                           (int32_t)((td - tb) | (te - td - 1) << 8 | local(jp[0]) << 16));
    rec[2 * p + 1] = make_int4(back[0], back[1], back[2], (int32_t)(local(jp[1]) | local(jp[2]) << 16));
    if (more) stats[0] = 1;
    if (back_by > 0) atomicMax(&far, back_by);
    __syncthreads();
    if (threadIdx.x == 0) atomicMax(&stats[1], far);
}

// Block ILU0 (Algorithm 5, IKJ order), the ILDU0 scaling and both sweeps'
// slot streams in one kernel, one workgroup per subdomain, levels of the
// lower sweep in turn; for patterns in which a lower block updates the pivot
// block only (7-point stencils in any numbering): L_IJ = A_IJ inv(U_JJ),
// U_II = A_II - sum_J L_IJ A_JI in ascending J, inv(U_II), Uhat_IK = inv(U_II)
// A_IK, the arithmetic of k_bilu0 followed by k_pack_slots, so the same bits.
// Between rows of one subdomain only the pivot inverses pass from level to
// level.
//
// A 3x3 row takes four lanes (the fourth repeats the third and stores
// nothing): lane c holds row c of every block, loads and stores 24
// contiguous bytes of it, and takes the other rows from its quad's lanes
// (quad_perm moves, no LDS).  All loads of a row are issued together,
// branch-free (positions past a row's end re-read its diagonal block), one
// chunk ahead.  The inverses pass through a ring in LDS by position (RING),
// so the barrier between levels waits for no memory access; where the rows
// reach too far back for the LDS they pass through invd.  One box alone takes
// 4.3 us a level of 16^3 (7.1 with the inverses through invd and nothing
// loaded ahead).  2,097,152 3x3 rows in 512 boxes of 16^3: 1,330 us with a
// copy of L and U in the dropped pattern, which few callers read (k_lu_blocks
// makes it for them), 913 without, 855 with the ring (then 877 with a word of
// each line fetched a chunk earlier, 843 with 4 wavefronts a box instead of
// 8), 796 with the next chunk's loads ahead of the level barriers.  Not the
// memory's bound: 1.7 GB read and 1.3 GB written are 3.8 TB/s.  The stores
// reach the L2 as 95 million requests of 14 bytes on average, a lane's three
// doubles of a row one by one (loads 20 million); the 206 registers of a lane
// leave one box to a CU, so 264 boxes (99x80x108) take two rounds, 501 us.
template <int Q>
__device__ __forceinline__ double quad_bcast(double v) {
    constexpr int P = Q * 0x55;  // quad_perm: lane Q of each four
    const int2 w = __builtin_bit_cast(int2, v);
    int2 r;
    r.x = __builtin_amdgcn_mov_dpp(w.x, P, 0xf, 0xf, true);
    r.y = __builtin_amdgcn_mov_dpp(w.y, P, 0xf, 0xf, true);
    return __builtin_bit_cast(double, r);
}

// v times the block whose row c lane c holds in b: t_j = sum_q v_q b_qj
template <int BS>
__device__ __forceinline__ void row_times(const double (&v)[BS], const double (&b)[BS], double (&t)[BS]) {
#pragma unroll
    for (int j = 0; j < BS; ++j) {
        t[j] = 0.0;
        if constexpr (BS == 1) {
            t[j] += v[0] * b[j];
        } else {
            t[j] += v[0] * quad_bcast<0>(b[j]);
            t[j] += v[1] * quad_bcast<1>(b[j]);
            t[j] += v[2] * quad_bcast<2>(b[j]);
        }
    }
}

// One row of the factorisation on its quad (or lane): everything it reads, and
// where its parts go.  dg: A's position of the diagonal block (the row's
// nlow lower and nupp upper blocks next to it), J: lower columns, back: A's
// position of A_JI or -1, lo/uo: row c of the row's slot blocks.
template <int BS, int MB>
struct FactorRow {
    int64_t gi, dg, J[MB];
    int32_t back[MB];
    int nlow, nupp;
    double *lo, *uo;
};

// Row c of a row's blocks of A: diagonal, lower, A_JI of the lower columns,
// upper (positions past the row's end re-read its diagonal block).
template <int BS, int MB>
struct FactorVals {
    double D[BS], a[MB][BS], t[MB][BS], b[MB][BS];
};

template <int BS>
__device__ __forceinline__ void load_row(const double *p, double (&v)[BS]) {
#pragma unroll
    for (int j = 0; j < BS; ++j) v[j] = p[j];
}

template <int BS, int MB>
__device__ __forceinline__ void factor_values(const FactorRow<BS, MB> &R, int c, const double *__restrict__ aval,
                                              FactorVals<BS, MB> &V) {
    constexpr int BB = BS * BS;
    load_row<BS>(aval + R.dg * BB + c * BS, V.D);
#pragma unroll
    for (int k = 0; k < MB; ++k) {
        load_row<BS>(aval + (k < R.nlow ? R.dg - R.nlow + k : R.dg) * BB + c * BS, V.a[k]);
        load_row<BS>(aval + (R.back[k] >= 0 ? (int64_t)R.back[k] : R.dg) * BB + c * BS, V.t[k]);
        load_row<BS>(aval + (k < R.nupp ? R.dg + 1 + k : R.dg) * BB + c * BS, V.b[k]);
    }
}

// Row c of the lower columns' pivot inverses.
template <int BS, int MB>
__device__ __forceinline__ void factor_pivots(const FactorRow<BS, MB> &R, int c, const double *invd,
                                              double (&iv)[MB][BS]) {
#pragma unroll
    for (int k = 0; k < MB; ++k) load_row<BS>(invd + (k < R.nlow ? R.J[k] : R.gi) * BS * BS + c * BS, iv[k]);
}

template <int BS, int MB>
__device__ __forceinline__ void factor_row(const FactorRow<BS, MB> &R, const FactorVals<BS, MB> &V,
                                           const double (&iv)[MB][BS], bool ok, int c, bool store, bool first,
                                           double *invd, int32_t *status, double (&ic)[BS]) {
    constexpr int BB = BS * BS;
    auto put = [&](double *p, const double (&v)[BS]) {
#pragma unroll
        for (int j = 0; j < BS; ++j) p[j] = v[j];
    };
    double D[BS];
#pragma unroll
    for (int j = 0; j < BS; ++j) D[j] = V.D[j];
#pragma unroll
    for (int k = 0; k < MB; ++k) {
        double L[BS], w[BS];
        row_times<BS>(V.a[k], iv[k], L);
        row_times<BS>(L, V.t[k], w);
        const bool in = k < R.nlow;
#pragma unroll
        for (int j = 0; j < BS; ++j) {
            L[j] = in ? L[j] : 0.0;
            D[j] = in && R.back[k] >= 0 ? D[j] - w[j] : D[j];
        }
        if (ok && store) put(R.lo + k * BS, L);
    }
    double piv[BB], inv[BB];
#pragma unroll
    for (int j = 0; j < BS; ++j) {
        if constexpr (BS == 1) {
            piv[0] = D[0];
        } else {
            piv[j] = quad_bcast<0>(D[j]);
            piv[BS + j] = quad_bcast<1>(D[j]);
            piv[2 * BS + j] = quad_bcast<2>(D[j]);
        }
    }
    if (!blk_inverse<BS>(piv, inv)) {
        if (ok && first) atomicMin(&status[2], (int32_t)R.gi);
#pragma unroll
        for (int e = 0; e < BB; ++e) inv[e] = (e % (BS + 1) == 0) ? 1.0 : 0.0;
    }
#pragma unroll
    for (int j = 0; j < BS; ++j) {  // row c of the inverse
        ic[j] = inv[j];
#pragma unroll
        for (int i = 1; i < BS; ++i) ic[j] = c == i ? inv[i * BS + j] : ic[j];
    }
#pragma unroll
    for (int k = 0; k < MB; ++k) {
        double u[BS];
        row_times<BS>(ic, V.b[k], u);
        const bool in = k < R.nupp;
#pragma unroll
        for (int j = 0; j < BS; ++j) u[j] = in ? u[j] : 0.0;
        if (ok && store) put(R.uo + k * BS, u);
    }
    if (ok && store) {
        put(R.uo + MB * BS, ic);
        put(invd + R.gi * BB + c * BS, ic);
    }
}

// LDS writes before it are seen by LDS reads after it; memory accesses stay
// in flight.
__device__ __forceinline__ void lds_barrier() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

template <int BS, int MB, bool RING>
__global__ __launch_bounds__(512) void k_bilu0_slots(int S, const int32_t *__restrict__ off,
                                                    const int32_t *__restrict__ lptr,
                                                    const uint64_t *__restrict__ desc, const int4 *__restrict__ rec,
                                                    const double *__restrict__ aval, double *invd,
                                                    double *__restrict__ lval, double *__restrict__ uval,
                                                    int32_t *status, int ring, int lp_at) {
    constexpr int BB = BS * BS, LR = BS == 3 ? 4 : 1, RPW = kWave / LR, NL = MB * BS, NU = (MB + 1) * BS;
    extern __shared__ double pivots[];  // RING: inverse of position p at p mod ring (a power of two)
    int32_t *lp = reinterpret_cast<int32_t *>(pivots + lp_at);  // the levels' first positions
    const int s = blockIdx.x;
    const int64_t base = (int64_t)s * S;
    const int32_t o = off[s];
    const int nl = off[s + 1] - o - 1;
    const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave, nw = blockDim.x / kWave;
    const int rl = lane / LR, c = min(lane % LR, BS - 1);
    const bool store = lane % LR < BS;
    for (int i = threadIdx.x; i <= nl; i += blockDim.x) lp[i] = lptr[o + i];
    __syncthreads();

    // A chunk: up to RPW rows of one level from position pb; this wavefront's
    // chunks follow each other level by level (l = nl: none left).
    struct Chunk {
        int l, pb;
    };
    auto settle = [&](Chunk k) -> Chunk {  // to the level that has the position, if this one does not
        while (k.l < nl && k.pb >= lp[k.l + 1]) {
            ++k.l;
            if (k.l < nl) k.pb = lp[k.l] + wave * RPW;
        }
        k.l = __builtin_amdgcn_readfirstlane(k.l);
        k.pb = __builtin_amdgcn_readfirstlane(k.pb);
        return k;
    };
    struct Record {
        int4 r0, r1;
        uint64_t d;
    };
    auto place = [&](const Chunk &k) -> int {  // a lane past the level's end repeats a row of it
        if (k.l >= nl) return 0;
        return k.pb + rl < lp[k.l + 1] ? k.pb + rl : lp[k.l];
    };
    auto fetch = [&](const Chunk &k) -> Record {
        const int64_t gp = base + place(k);
        return Record{rec[2 * gp], rec[2 * gp + 1], desc[gp]};
    };
    auto row = [&](const Chunk &k, const Record &q) -> FactorRow<BS, MB> {
        FactorRow<BS, MB> R;
        R.nlow = q.r0.w & 0xff;
        R.nupp = q.r0.w >> 8 & 0xff;
        R.gi = base + (int)(q.d & 0xffff);
        R.dg = q.r0.x + R.nlow;
        const int32_t back[3] = {q.r1.x, q.r1.y, q.r1.z};
#pragma unroll
        for (int j = 0; j < MB; ++j) {
            R.J[j] = base + (int)((q.d >> (16 * (j + 1))) & 0xffff);
            R.back[j] = back[j];
        }
        R.lo = lval + ((base + place(k)) * BS + c) * NL;
        R.uo = uval + ((int64_t)q.r0.z * BS + c) * NU;
        return R;
    };
    int lev = 0;  // barriers passed
    Chunk k0 = settle({0, wave * RPW}), k1 = settle({k0.l, k0.pb + nw * RPW});
    Record q0 = fetch(k0), q1 = fetch(k1);
    FactorVals<BS, MB> va, vb;
    factor_values<BS, MB>(row(k0, q0), c, aval, va);
    // one chunk from v; next: the set for the following chunk's blocks
    auto step = [&](const FactorVals<BS, MB> &v, FactorVals<BS, MB> &next) {
        // in flight before the barriers: what does not depend on the levels
        const Chunk k2 = settle({k1.l, k1.pb + nw * RPW});
        const Record q2 = fetch(k2);
        factor_values<BS, MB>(row(k1, q1), c, aval, next);
        __builtin_amdgcn_sched_barrier(0);
        for (; lev < k0.l; ++lev) {
            if constexpr (RING)
                lds_barrier();
            else
                __syncthreads();
        }
        const FactorRow<BS, MB> R = row(k0, q0);
        double iv[MB][BS];
        if constexpr (RING) {
            const int jp[3] = {(int)((uint32_t)q0.r0.w >> 16), q0.r1.w & 0xffff, (int)((uint32_t)q0.r1.w >> 16)};
#pragma unroll
            for (int j = 0; j < MB; ++j) load_row<BS>(pivots + ((jp[j] & (ring - 1)) * BB + c * BS), iv[j]);
        } else {
            factor_pivots<BS, MB>(R, c, invd, iv);
        }
        const bool ok = k0.pb + rl < lp[k0.l + 1];
        double ic[BS];
        factor_row<BS, MB>(R, v, iv, ok, c, store, lane % LR == 0, invd, status, ic);
        if constexpr (RING) {
            if (ok && store) {
#pragma unroll
                for (int j = 0; j < BS; ++j) pivots[((k0.pb + rl) & (ring - 1)) * BB + c * BS + j] = ic[j];
            }
        }
        k0 = k1;
        k1 = k2;
        q0 = q1;
        q1 = q2;
    };
    while (k0.l < nl) {
        step(va, vb);
        if (k0.l >= nl) break;
        step(vb, va);
    }
    for (; lev < nl; ++lev) {
        if constexpr (RING)
            lds_barrier();
        else
            __syncthreads();
    }
}

// The same for the rows of one level of the undecomposed matrix (global ILU0):
// records {row, A's diagonal position, nlow | nupp << 8, lower-sweep
// position}, {J0, J1, J2, upper-sweep position}, {A's positions of A_JI, 0} in level order;
// three slots.
template <int BS>
__global__ __launch_bounds__(256) void k_gfactor_slots(int32_t p0, int32_t p1, const int4 *__restrict__ rec,
                                                      const double *__restrict__ aval, double *invd,
                                                      double *__restrict__ lval, double *__restrict__ uval,
                                                      int32_t *status) {
    constexpr int LR = BS == 3 ? 4 : 1, MB = kMaxSlots;
    const int lane = threadIdx.x & (kWave - 1), c = min(lane % LR, BS - 1);
    const int32_t p = p0 + (int32_t)(((int64_t)blockIdx.x * blockDim.x + threadIdx.x) / LR);
    const bool ok = p < p1;
    const int64_t q = 3 * (int64_t)(ok ? p : p0);
    const int4 r0 = rec[q], r1 = rec[q + 1], r2 = rec[q + 2];
    FactorRow<BS, MB> R;
    R.gi = r0.x;
    R.dg = r0.y;
    R.nlow = r0.z & 0xff;
    R.nupp = r0.z >> 8;
    R.J[0] = r1.x; R.J[1] = r1.y; R.J[2] = r1.z;
    R.back[0] = r2.x; R.back[1] = r2.y; R.back[2] = r2.z;
    R.lo = lval + ((int64_t)r0.w * BS + c) * MB * BS;
    R.uo = uval + ((int64_t)r1.w * BS + c) * (MB + 1) * BS;
    FactorVals<BS, MB> V;
    double iv[MB][BS], ic[BS];
    factor_values<BS, MB>(R, c, aval, V);
    factor_pivots<BS, MB>(R, c, invd, iv);
    __builtin_amdgcn_sched_barrier(0);
    factor_row<BS, MB>(R, V, iv, ok, c, lane % LR < BS, lane % LR == 0, invd, status, ic);
}

// One launch per level of the lower sweep (host offsets lp[0..nlev]).
hipError_t launch_gfactor_slots(dd_ctx *h, const std::vector<int32_t> &lp, hipStream_t st) {
    const int lr = h->bs == 3 ? 4 : 1;
    for (size_t l = 0; l + 1 < lp.size(); ++l) {
        const unsigned g = (unsigned)(((int64_t)(lp[l + 1] - lp[l]) * lr + 255) / 256);
        if (h->bs == 3)
            k_gfactor_slots<3><<<g, 256, 0, st>>>(lp[l], lp[l + 1], h->grec, h->aval, h->ginvd, h->gsval[0],
                                                  h->gsval[1], h->status);
        else
            k_gfactor_slots<1><<<g, 256, 0, st>>>(lp[l], lp[l + 1], h->grec, h->aval, h->ginvd, h->gsval[0],
                                                  h->gsval[1], h->status);
    }
    return hipGetLastError();
}

hipError_t launch_slot_records(dd_ctx *h, int32_t *stats, hipStream_t st) {
    const int T = 256;
    const unsigned g = (unsigned)((h->n + T - 1) / T);
    k_slot_desc<<<dim3(g, 2), T, 0, st>>>(h->n, h->S, h->tptr, h->tcol, h->tdiag, h->lev[0].rows, h->lev[1].rows,
                                          h->sw[0].desc, h->sw[1].desc);
    k_factor_records<<<g, T, 0, st>>>(h->n, h->S, h->tptr, h->tcol, h->tdiag, h->tsrc, h->lev[0].rows, h->linv,
                                      h->uinv, h->frec, stats);
    return hipGetLastError();
}

hipError_t launch_bilu0_slots(dd_ctx *h, hipStream_t st) {
    const Levels &L = h->lev[0];
    const int rpw = h->bs == 3 ? kWave / 4 : kWave;
    int waves = 1;  // for the widest level, at most 8
    while (waves < 8 && waves * rpw < h->max_level_width) waves *= 2;
    // The ring holds a row's inverse until every row that reads it is done: no
    // row reads further back than the records found, and the rows of one
    // level are written in any order.
    const size_t lp = (size_t)(L.max_levels + 1) * sizeof(int32_t), one = (size_t)h->bs * h->bs * sizeof(double);
    int ring = 1;
    while (ring < h->reach + h->max_level_width) ring *= 2;
    const bool in_lds = ring * one + lp <= 163840 - 1024;
    const size_t lds = (in_lds ? ring * one : 0) + lp;
    auto go = [&](auto kern) {
        if (lds > 65536) (void)full_lds(kern);
        kern<<<h->nsub, waves * kWave, lds, st>>>(h->S, L.off, L.ptr, h->sw[0].desc, h->frec, h->aval, h->invd,
                                                h->sw[0].sval64, h->sw[1].sval64, h->status, ring,
                                                in_lds ? ring * h->bs * h->bs : 0);
    };
    auto pick = [&](auto bs, auto mb) {
        if (in_lds)
            go(k_bilu0_slots<decltype(bs)::value, decltype(mb)::value, true>);
        else
            go(k_bilu0_slots<decltype(bs)::value, decltype(mb)::value, false>);
    };
    auto slots = [&](auto bs) {
        if (h->slots == 1)
            pick(bs, std::integral_constant<int, 1>{});
        else if (h->slots == 2)
            pick(bs, std::integral_constant<int, 2>{});
        else
            pick(bs, std::integral_constant<int, 3>{});
    };
    if (h->bs == 3)
        slots(std::integral_constant<int, 3>{});
    else
        slots(std::integral_constant<int, 1>{});
    return hipGetLastError();
}

// L and U in the dropped pattern, from the streams and the matrix (the
// patterns of k_bilu0_slots leave U's off-diagonal blocks as A's): for the
// CSR streams and the adjoint streams.  Their diagonal blocks are
// inv_D's, so lu's are not written.  Written with every factorisation, the
// copy was 1.1 of its 2.3 GB of stores (2,097,152 3x3 rows).
template <int BS>
__global__ __launch_bounds__(256) void k_lu_blocks(int64_t n, int MB, const int4 *__restrict__ rec,
                                                  const double *__restrict__ aval, const double *__restrict__ lval,
                                                  double *__restrict__ lu) {
    constexpr int BB = BS * BS;
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int64_t p = t / (2 * MB);
    if (p >= n) return;
    const int j = (int)(t - p * 2 * MB), k = j < MB ? j : j - MB;
    const int4 r = rec[2 * p];
    const int nlow = r.w & 0xff, nupp = r.w >> 8 & 0xff;
    if (k >= (j < MB ? nlow : nupp)) return;
    const int at = j < MB ? k : nlow + 1 + k;
#pragma unroll
    for (int e = 0; e < BB; ++e)
        lu[(int64_t)(r.y + at) * BB + e] = j < MB ? lval[(p * BS + e / BS) * MB * BS + k * BS + e % BS]
                                                  : aval[(int64_t)(r.x + at) * BB + e];
}

hipError_t launch_lu_blocks(dd_ctx *h, hipStream_t st) {
    if (!h->direct) return hipSuccess;  // the factorisation left them
    const unsigned g = (unsigned)((h->n * 2 * h->slots + 255) / 256);
    if (h->bs == 3)
        k_lu_blocks<3><<<g, 256, 0, st>>>(h->n, h->slots, h->frec, h->aval, h->sw[0].sval64, h->lu);
    else
        k_lu_blocks<1><<<g, 256, 0, st>>>(h->n, h->slots, h->frec, h->aval, h->sw[0].sval64, h->lu);
    return hipGetLastError();
}

// The factors in the dropped pattern (see dd_get_factors) from the streams,
// which hold them in that form; one thread per value a row can have, so a
// row's blocks are written as one run.  64^3 3x3 blocks: 334 us with L and U made
// first (k_lu_blocks, k_export), 112 with L and U at hand, 79 like this.
template <int BS>
__global__ __launch_bounds__(256) void k_export_slots(int64_t n, int MB, const int4 *__restrict__ rec,
                                                     const double *__restrict__ lval,
                                                     const double *__restrict__ uval, double *__restrict__ f) {
    constexpr int BB = BS * BS;
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int row = (2 * MB + 1) * BB;
    const int64_t p = t / row;
    if (p >= n) return;
    const int q = (int)(t - p * row), j = q / BB, e = q - j * BB;
    const int4 r = rec[2 * p];
    const int nlow = r.w & 0xff, nupp = r.w >> 8 & 0xff;
    if (j >= nlow + 1 + nupp) return;
    // lower blocks, inv_D (the upper stream's last slot), upper blocks
    const int k = j == nlow ? MB : j - nlow - 1;
    f[(int64_t)r.y * BB + q] = j < nlow ? lval[(p * BS + e / BS) * MB * BS + j * BS + e % BS]
                                        : uval[((int64_t)r.z * BS + e / BS) * (MB + 1) * BS + k * BS + e % BS];
}

hipError_t launch_export_slots(dd_ctx *h, double *f, hipStream_t st) {
    const int64_t threads = h->n * (2 * h->slots + 1) * h->bs * h->bs;
    const unsigned g = (unsigned)((threads + 255) / 256);
    if (h->bs == 3)
        k_export_slots<3><<<g, 256, 0, st>>>(h->n, h->slots, h->frec, h->sw[0].sval64, h->sw[1].sval64, f);
    else
        k_export_slots<1><<<g, 256, 0, st>>>(h->n, h->slots, h->frec, h->sw[0].sval64, h->sw[1].sval64, f);
    return hipGetLastError();
}

// ------------------------------------------------- segmented slot layout
// For sweeps with rows of more than three blocks.  With MB blocks per
// segment, a lower-sweep row with nb blocks becomes ceil(nb/MB) segments (none
// when nb = 0: y_I = r_I), an upper-sweep row one segment of MB blocks and
// inv_D plus ceil((nb - MB)/(MB + 1)) continuations of MB + 1 blocks (the
// extra block in the inv_D slot, which a continuation does not need); blocks
// in column order, segments at consecutive positions; the first segment (the
// row's owner) adds the others' partial sums in the apply, by cross-lane reads:
// so a wave-chunk takes whole rows, as many as fit its positions.  Positions
// follow each other without padding (chunks name their own extent), the
// streams are the sum of the segments.
__device__ __forceinline__ int seg_count(int which, int nb, int mb) {
    return which == 0 ? (nb + mb - 1) / mb : 1 + (max(nb - mb, 0) + mb) / (mb + 1);
}

// positions of each subdomain (blockIdx.y = sweep)
__global__ __launch_bounds__(256) void k_seg_count(int S, int mb, const int32_t *__restrict__ tptr,
                                                  const int32_t *__restrict__ tcol,
                                                  const int32_t *__restrict__ tdiag, int32_t *__restrict__ npos0,
                                                  int32_t *__restrict__ npos1) {
    __shared__ int sum;
    const int which = blockIdx.y, s = blockIdx.x;
    const int64_t base = (int64_t)s * S;
    if (threadIdx.x == 0) sum = 0;
    __syncthreads();
    int m = 0;
    for (int i = threadIdx.x; i < S; i += blockDim.x) {
        int32_t lo, hi;
        dep_range(which, base + i, tptr, tcol, tdiag, lo, hi);
        m += seg_count(which, hi - lo, mb);
    }
    atomicAdd(&sum, m);
    __syncthreads();
    if (threadIdx.x == 0) (which ? npos1 : npos0)[s] = sum;
}

// Position map and wave-chunks of each subdomain (one workgroup each, y =
// sweep): a scan over the rows in sweep order gives every row's first
// position; then one wavefront cuts each level, finding by ballot how many
// rows the next chunk holds.  wbase bounds the chunks before: all but a
// level's last hold more than rpw - kSegMax positions.  Placing the rows one
// by one in one thread: 2 x 2 x 555 us for 1,024,000 rows in 250 parts; 60 us.
__global__ __launch_bounds__(512) void k_seg_fill(int S, int mb, int rpw, const int32_t *__restrict__ tptr,
                                                 const int32_t *__restrict__ tcol,
                                                 const int32_t *__restrict__ tdiag, const int32_t *__restrict__ off0,
                                                 const int32_t *__restrict__ off1, const int32_t *__restrict__ lp0,
                                                 const int32_t *__restrict__ lp1, const int32_t *__restrict__ rows0,
                                                 const int32_t *__restrict__ rows1,
                                                 const int32_t *__restrict__ gpos0,
                                                 const int32_t *__restrict__ gpos1, int2 *__restrict__ pmap0,
                                                 int2 *__restrict__ pmap1, int2 *__restrict__ wtab0,
                                                 int2 *__restrict__ wtab1, int4 *__restrict__ winfo0,
                                                 int4 *__restrict__ winfo1) {
    extern __shared__ int32_t first[];  // [S + 1] first position of each row in sweep order
    __shared__ int sh[65];
    const int which = blockIdx.y, s = blockIdx.x, tid = threadIdx.x, nt = blockDim.x;
    const int64_t base = (int64_t)s * S;
    const int32_t *rows = which ? rows1 : rows0;
    const int32_t g0 = (which ? gpos1 : gpos0)[s];
    int2 *pmap = (which ? pmap1 : pmap0) + g0;
    int done = 0;
    for (int t0 = 0; t0 < S; t0 += nt) {
        const int i = t0 + tid;
        int m = 0;
        int64_t gi = 0;
        if (i < S) {
            gi = base + rows[base + i];
            int32_t lo, hi;
            dep_range(which, gi, tptr, tcol, tdiag, lo, hi);
            m = seg_count(which, hi - lo, mb);
        }
        int tot;
        const int at = done + block_excl_scan(m, sh, &tot);
        if (i < S) first[i] = at;
        for (int q = 0; q < m; ++q) pmap[at + q] = make_int2((int32_t)gi, q | m << 8);
        done += tot;
    }
    if (tid == 0) first[S] = done;
    __syncthreads();
    if (tid >= kWave) return;
    const int32_t o = (which ? off1 : off0)[s];
    const int nl = (which ? off1 : off0)[s + 1] - o - 1;
    const int32_t *lp = (which ? lp1 : lp0) + o;
    const int32_t wbase = g0 / (rpw - kSegMax + 1) + s + o;
    int2 *wtab = (which ? wtab1 : wtab0) + wbase;
    int chunks = 0, level = 0;  // levels without positions (the lower sweep's first) are not counted
    for (int l = 0; l < nl; ++l) {
        const int e = lp[l + 1], before = chunks;
        for (int i = lp[l]; i < e;) {
            const int p0 = first[i];
            for (int c = kWave; c == kWave;) {
                const int j = i + 1 + tid;
                c = __popcll(__ballot(j <= e && first[min(j, S)] - p0 <= rpw));
                i += c;  // at least one row: a row has at most kSegMax segments
            }
            const int cnt = first[i] - p0;
            if (cnt == 0) continue;
            if (tid == 0) wtab[chunks] = make_int2(p0, level << 8 | cnt);
            ++chunks;
        }
        level += chunks > before ? 1 : 0;
    }
    if (tid == 0) (which ? winfo1 : winfo0)[s] = make_int4(wbase, chunks, level, 0);
}

// Position p: its segment's descriptor and values in the lane-run layout of
// k_pack_slots (MB blocks, then inv_D in the upper sweep), from the factors
// in the dropped pattern, Uhat = inv_D U on the way.  Lanes as in factor_row:
// a quad per 3x3 position, lane c its blocks' row c, so stores are whole
// runs.  An upper-sweep continuation holds its (MB+1)-th block in the inv_D
// slot and that block's column in the row field (its own row when the slot is
// empty: a valid LDS entry, times a zero block).  The descriptor keeps three
// 16-bit column fields whatever MB (fields past MB empty), so that the bits 15
// of fields 1 to 3 hold m - 1 on a row's first segment.
template <int BS, int MB, int WHICH>
__global__ __launch_bounds__(256) void k_seg_pack(int64_t npos, int S, const int2 *__restrict__ pmap,
                                                 const int32_t *__restrict__ tptr, const int32_t *__restrict__ tcol,
                                                 const int32_t *__restrict__ tdiag, const double *__restrict__ lu,
                                                 const double *__restrict__ invd, uint64_t *__restrict__ desc,
                                                 double *__restrict__ sval) {
    constexpr int BB = BS * BS, LR = BS == 3 ? 4 : 1, NV = (MB + WHICH) * BS;
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int64_t p = t / LR;
    const int l = (int)(t % LR), c = min(l, BS - 1);
    const bool ok = p < npos;
    const int2 e = pmap[ok ? p : 0];
    const int k = e.y & 0xff, m = e.y >> 8;
    const int64_t gi = e.x, base = gi / S * S;
    int32_t lo, hi;
    dep_range(WHICH, gi, tptr, tcol, tdiag, lo, hi);
    const int32_t b0 = lo + (WHICH == 0 || k == 0 ? MB * k : MB + (k - 1) * (MB + 1));
    const int32_t b1 = min(b0 + MB, hi);
    const int32_t bx = WHICH == 1 && k > 0 && b0 + MB < hi ? b0 + MB : -1;  // a continuation's extra block
    double iv[BS];
#pragma unroll
    for (int j = 0; j < BS; ++j) iv[j] = WHICH == 1 ? invd[gi * BB + c * BS + j] : 0.0;
    double *o = sval + (p * BS + c) * NV;
#pragma unroll
    for (int q = 0; q < MB + WHICH; ++q) {
        const int32_t b = q < MB ? (b0 + q < b1 ? b0 + q : -1) : bx;
        double v[BS], u[BS];
#pragma unroll
        for (int j = 0; j < BS; ++j) v[j] = b >= 0 ? lu[(int64_t)b * BB + c * BS + j] : 0.0;
        if constexpr (WHICH == 1) {
            row_times<BS>(iv, v, u);
#pragma unroll
            for (int j = 0; j < BS; ++j) v[j] = q == MB && k == 0 ? iv[j] : (b >= 0 ? u[j] : 0.0);
        }
        if (ok && l < BS)
#pragma unroll
            for (int j = 0; j < BS; ++j) o[q * BS + j] = v[j];
    }
    if (!ok || l != 0) return;
    uint64_t d = (uint64_t)(bx >= 0 ? tcol[bx] - (int32_t)base : (int32_t)(gi - base)) | (k > 0 ? 0x8000ull : 0ull);
    for (int j = 0; j < 3; ++j)
        d |= (uint64_t)(j < MB && b0 + j < b1 ? tcol[b0 + j] - (int32_t)base : 0x7fff) << (16 * (j + 1));
    if (k == 0)
        for (int j = 0; j < 3; ++j)
            if (((m - 1) >> j) & 1) d |= 1ull << (16 * (j + 1) + 15);
    desc[p] = d;
}

hipError_t launch_seg_pack(dd_ctx *h, hipStream_t st) {
    const int lr = h->bs == 3 ? 4 : 1;
    for (int w = 0; w < 2; ++w) {
        Sweep &s = h->sw[w];
        if (s.snpos == 0) continue;
        const unsigned g = (unsigned)((s.snpos * lr + 255) / 256);
        auto go = [&](auto kern) {
            kern<<<g, 256, 0, st>>>(s.snpos, h->S, s.pmap, h->tptr, h->tcol, h->tdiag, h->lu, h->invd, s.desc,
                                    s.sval64);
        };
        switch ((h->bs == 3 ? 0 : 4) + (h->seg == 2 ? 0 : 2) + w) {
            case 0: go(k_seg_pack<3, 2, 0>); break;
            case 1: go(k_seg_pack<3, 2, 1>); break;
            case 2: go(k_seg_pack<3, 3, 0>); break;
            case 3: go(k_seg_pack<3, 3, 1>); break;
            case 4: go(k_seg_pack<1, 2, 0>); break;
            case 5: go(k_seg_pack<1, 2, 1>); break;
            case 6: go(k_seg_pack<1, 3, 0>); break;
            default: go(k_seg_pack<1, 3, 1>); break;
        }
    }
    return hipGetLastError();
}

// Positions, chunks and values of both sweeps (h->seg set).
int build_seg_layout(dd_ctx *h, hipStream_t st) {
    const int mb = h->seg, rpw = kWave / h->bs, bb = h->bs * h->bs, nsub = h->nsub;
    int32_t *npos[2] = {nullptr, nullptr}, tot[2] = {0, 0};
    int rc = DD_OK;
    for (int w = 0; w < 2 && !rc; ++w) {
        rc = h->alloc(&npos[w], nsub);
        if (!rc && !h->sw[w].gpos) rc = h->alloc(&h->sw[w].gpos, nsub + 1);
    }
    if (rc) return rc;
    k_seg_count<<<dim3(nsub, 2), 256, 0, st>>>(h->S, mb, h->tptr, h->tcol, h->tdiag, npos[0], npos[1]);
    hipError_t e = hipGetLastError();
    for (int w = 0; w < 2; ++w) {
        if (e == hipSuccess) e = exclusive_scan(npos[w], h->sw[w].gpos, nsub, h->scan_tmp, st);
        if (e == hipSuccess)
            e = hipMemcpyAsync(&tot[w], h->sw[w].gpos + nsub, sizeof(int32_t), hipMemcpyDeviceToHost, st);
    }
    if (e == hipSuccess) e = hipStreamSynchronize(st);
    if (e != hipSuccess) return h->fail(DD_EHIP, "segmented layout: %s", hipGetErrorString(e));
    for (int w = 0; w < 2 && !rc; ++w) {
        Sweep &s = h->sw[w];
        h->release(s.pmap);
        h->release(s.wtab);
        h->release(s.winfo);
        h->release(npos[w]);
        s.snpos = tot[w];
        rc = h->alloc(&s.pmap, tot[w]);
        if (!rc) rc = h->alloc(&s.wtab, tot[w] / (rpw - kSegMax + 1) + nsub + h->lev[w].ptr_len + 1);
        if (!rc) rc = h->alloc(&s.winfo, nsub);
        if (!rc) rc = h->alloc(&s.desc, tot[w]);
        if (!rc) rc = h->alloc(&s.sval64, (int64_t)tot[w] * (mb + w) * bb);
    }
    if (rc) return rc;
    Sweep &L = h->sw[0], &U = h->sw[1];
    e = full_lds(k_seg_fill);
    if (e == hipSuccess) {
        k_seg_fill<<<dim3(nsub, 2), 512, (size_t)(h->S + 1) * sizeof(int32_t), st>>>(
            h->S, mb, rpw, h->tptr, h->tcol, h->tdiag, h->lev[0].off, h->lev[1].off, h->lev[0].ptr, h->lev[1].ptr,
            h->lev[0].rows, h->lev[1].rows, L.gpos, U.gpos, L.pmap, U.pmap, L.wtab, U.wtab, L.winfo, U.winfo);
        e = hipGetLastError();
    }
    if (e == hipSuccess) e = launch_seg_pack(h, st);
    if (e != hipSuccess) return h->fail(DD_EHIP, "segmented layout: %s", hipGetErrorString(e));
    return DD_OK;
}

}  // namespace ddilu
