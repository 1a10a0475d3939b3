// Partition labels for a matrix graph without geometry (Section 3: labels
// from a graph partitioner; Section 5.3: parts balanced to one size), as a
// stand-in for METIS: recursive BFS bisection into parts of exactly S
// vertices.  A segment of k parts (k*S vertices, all labelled with its first
// part number b) splits, if k > 1, by a BFS inside the segment from its
// smallest vertex, a second BFS from the reached vertex of largest distance
// (smallest index on ties), and the order (distance, index) with unreached
// vertices last: the first floor(k/2)*S vertices keep label b, the rest take
// b + floor(k/2).  Every segment of one depth is processed at once: the BFS
// levels relax all segments together (edges between segments are ignored),
// and one stable radix sort of (label, distance) keys orders all segments.
// After the last depth, the labels are the part numbers, and the vertices
// are renumbered by a stable sort on the label (Algorithm 3's order).
#include <hipcub/hipcub.hpp>

#include "blocks.h"
#include "internal.h"

namespace ddilu {

namespace {

constexpr uint32_t kInf = 0xffffffffu;
constexpr int kT = 256;
constexpr int kLevelBatch = 16;  // BFS levels launched between checks for progress

inline unsigned blocks(int64_t n) { return (unsigned)((n + kT - 1) / kT); }

__global__ void k_gp_fill(int64_t n, int32_t *a, int32_t v) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) a[i] = v;
}

__global__ void k_gp_fill64(int64_t n, unsigned long long *a) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) a[i] = 0ull;
}

// Per segment that splits at this depth: its smallest vertex (FAR = false), or
// the reached vertex of largest distance, smallest index on ties, as a key.
// A workgroup reduces its vertices into an LDS table over the labels and
// adds each entry to the global one once: one atomic per vertex on the few
// addresses of the first depths took 1,000 and 770 us at 1M vertices.
constexpr int kTable = 4096;  // labels the LDS table holds

template <bool FAR>
__global__ __launch_bounds__(1024) void k_gp_extreme(int64_t n, int32_t nparts, const int32_t *__restrict__ label,
                                                    const int32_t *__restrict__ segk,
                                                    const uint32_t *__restrict__ dist, int32_t *src,
                                                    unsigned long long *far) {
    __shared__ unsigned long long best[kTable];
    const bool table = nparts <= kTable;
    for (int b = threadIdx.x; table && b < nparts; b += blockDim.x) best[b] = 0;
    __syncthreads();
    // larger is better: the complement of the index, behind the distance
    for (int64_t v = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; v < n; v += (int64_t)gridDim.x * blockDim.x) {
        const int32_t b = label[v];
        const uint32_t d = FAR ? dist[v] : 0;
        if (segk[b] <= 1 || (FAR && d == kInf)) continue;
        const unsigned long long key = ((unsigned long long)d << 32) | (unsigned long long)(~(uint32_t)v);
        if (table) {
            if (key > best[b]) atomicMax(&best[b], key);
        } else if constexpr (FAR) {
            if (key > far[b]) atomicMax(&far[b], key);
        } else {
            if ((int32_t)v < src[b]) atomicMin(&src[b], (int32_t)v);
        }
    }
    __syncthreads();
    for (int b = threadIdx.x; table && b < nparts; b += blockDim.x) {
        if (!best[b]) continue;
        if constexpr (FAR)
            atomicMax(&far[b], best[b]);
        else
            atomicMin(&src[b], (int32_t)~(uint32_t)(best[b] & 0xffffffffull));
    }
}

__global__ void k_gp_src(int64_t n, const int32_t *label, const int32_t *segk, const int32_t *src,
                         uint32_t *dist) {
    const int64_t v = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (v >= n) return;
    const int32_t b = label[v];
    dist[v] = (segk[b] > 1 && src[b] == (int32_t)v) ? 0u : kInf;
}

// one BFS level: the vertices at distance d reach their unvisited neighbours
// of the same segment (every writer stores the same d + 1).  Few vertices are
// at d, so a level costs a launch and the latency of one vertex: its neighbours
// are read kNb at a time, all labels and distances of a batch in flight
// together (one neighbour after another: 14 us a level at 1M vertices), and a
// workgroup collects the vertices at d among kPer distances per thread before
// it follows them, which takes a quarter of the workgroups (one distance per
// thread 6.9 us a level, four 5.9, eight 6.0).
constexpr int kNb = 8;
constexpr int kPer = 4;  // distances a thread reads

__global__ __launch_bounds__(kT) void k_gp_level(int64_t n, const int32_t *__restrict__ ptr,
                                                const int32_t *__restrict__ col, const int32_t *__restrict__ label,
                                                uint32_t d, uint32_t *dist, int32_t *changed) {
    __shared__ int32_t list[kPer * kT];
    __shared__ int count;
    if (threadIdx.x == 0) count = 0;
    const int64_t v0 = kPer * ((int64_t)blockIdx.x * blockDim.x + threadIdx.x);
    uint32_t dv[kPer];
    if (v0 + kPer <= n) {
#pragma unroll
        for (int j = 0; j < kPer; j += 4) {
            const uint4 t = *reinterpret_cast<const uint4 *>(dist + v0 + j);
            dv[j] = t.x;
            dv[j + 1] = t.y;
            dv[j + 2] = t.z;
            dv[j + 3] = t.w;
        }
    } else {
#pragma unroll
        for (int j = 0; j < kPer; ++j) dv[j] = v0 + j < n ? dist[v0 + j] : kInf;
    }
    __syncthreads();
#pragma unroll
    for (int j = 0; j < kPer; ++j)
        if (dv[j] == d) list[atomicAdd(&count, 1)] = (int32_t)(v0 + j);
    __syncthreads();
    bool any = false;
    for (int i = threadIdx.x; i < count; i += kT) {
        const int32_t v = list[i], b = label[v], q0 = ptr[v], q1 = ptr[v + 1];
        for (int32_t q = q0; q < q1; q += kNb) {
            int32_t u[kNb], lu[kNb];
            uint32_t du[kNb];
#pragma unroll
            for (int j = 0; j < kNb; ++j) u[j] = col[min(q + j, q1 - 1)];
#pragma unroll
            for (int j = 0; j < kNb; ++j) {
                lu[j] = label[u[j]];
                du[j] = dist[u[j]];
            }
#pragma unroll
            for (int j = 0; j < kNb; ++j)
                if (lu[j] == b && du[j] == kInf) {
                    dist[u[j]] = d + 1;
                    any = true;
                }
        }
    }
    if (any) *changed = 1;
}

__global__ void k_gp_far_src(int32_t nparts, const int32_t *segk, const unsigned long long *far, int32_t *src) {
    const int32_t b = blockIdx.x * blockDim.x + threadIdx.x;
    if (b < nparts && segk[b] > 1) src[b] = (int32_t)(~(uint32_t)(far[b] & 0xffffffffull));
}

__global__ void k_gp_keys(int64_t n, const int32_t *label, const uint32_t *dist, unsigned long long *key,
                          int32_t *idx) {
    const int64_t v = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (v >= n) return;
    key[v] = ((unsigned long long)(uint32_t)label[v] << 32) | dist[v];
    idx[v] = (int32_t)v;
}

// the segment of label b starts at sorted position b*S: every smaller label
// heads a segment whose vertices all come first
__global__ void k_gp_split(int64_t n, int32_t S, const int32_t *sorted, const int32_t *segk, int32_t *label) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const int32_t v = sorted[i];
    const int32_t b = label[v];
    const int32_t k = segk[b];
    if (k <= 1) return;
    const int32_t k0 = k / 2;
    label[v] = (i - (int64_t)b * S) < (int64_t)k0 * S ? b : b + k0;
}

__global__ void k_gp_label_keys(int64_t n, const int32_t *label, uint32_t *key, int32_t *idx) {
    const int64_t v = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (v >= n) return;
    key[v] = (uint32_t)label[v];
    idx[v] = (int32_t)v;
}

__global__ void k_gp_perm(int64_t n, const int32_t *sorted, int32_t *new2old, int32_t *old2new) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const int32_t v = sorted[i];
    new2old[i] = v;
    old2new[v] = (int32_t)i;
}

__global__ void k_gp_pos(int64_t n, const int32_t *__restrict__ vlist, int32_t *__restrict__ pos) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) pos[vlist[i]] = (int32_t)i;
}

__global__ void k_gp_iota(int64_t n, int32_t *__restrict__ a, int32_t *__restrict__ b) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) a[i] = b[i] = (int32_t)i;
}

// One split of a segment of at most kLocal vertices, whole, in one workgroup:
// distances and the BFS queue in LDS, the segment's adjacency as local numbers
// in memory (0xffff: another segment).  vlist holds the segment's vertices
// at b*S .. (in any order), pos its inverse.  The queue's level boundaries
// give the distance at which the first floor(k/2)*S vertices end; of that
// distance (or of the unreached vertices) those of smallest index belong to
// them, found by bisection on the index.  Replaces, for the last depths, two
// BFS of one launch a level over all vertices, a sort and a relabelling.
constexpr int kLocal = 36864;  // dist and queue (2 + 2 bytes), visited bits: 152 KB
constexpr int kLocalT = 1024;

__host__ __device__ constexpr int local_lds(int len) { return (len + 31) / 32 * 32 * 4 + (len + 31) / 32 * 4; }

// k_gp_adj makes that adjacency for the segments that split, one thread per
// vertex, `per` workgroups a segment (vlist is written for these only): the
// scattered reads need more than one CU per segment (1M vertices in segments
// of 32 K to 8 K: 1,279 us a depth inside k_gp_local, 163 + 750 apart).  vlist
// holds every segment as one run of positions, so a neighbour's position tells
// its segment.
__global__ __launch_bounds__(kT) void k_gp_adj(int32_t S, int per, const int32_t *__restrict__ seg,
                                              const int32_t *__restrict__ segk, const int32_t *__restrict__ ptr,
                                              const int32_t *__restrict__ col,
                                              const int32_t *__restrict__ vlist, const int32_t *__restrict__ pos,
                                              uint16_t *__restrict__ ladj, int2 *__restrict__ range) {
    const int32_t b = seg[blockIdx.x / per];
    const uint32_t base = (uint32_t)b * S, len = (uint32_t)segk[b] * S;  // the segment's positions
    const uint32_t at = (blockIdx.x % per) * kT + threadIdx.x;
    if (at >= len) return;
    const int64_t i = (int64_t)base + at;
    const int32_t v = vlist[i], q0 = ptr[v], q1 = ptr[v + 1];
    range[i] = make_int2(q0, q1);
    for (int32_t q = q0; q < q1; q += kNb) {
        int32_t u[kNb];
        uint32_t l[kNb];
#pragma unroll
        for (int j = 0; j < kNb; ++j) u[j] = col[min(q + j, q1 - 1)];
#pragma unroll
        for (int j = 0; j < kNb; ++j) l[j] = (uint32_t)pos[u[j]] - base;
#pragma unroll
        for (int j = 0; j < kNb; ++j)
            if (q + j < q1) ladj[q + j] = l[j] < len ? (uint16_t)l[j] : 0xffff;
    }
}

__global__ __launch_bounds__(kLocalT) void k_gp_local(int32_t S, const int32_t *__restrict__ seg,
                                                     const int32_t *__restrict__ segk, int32_t *label,
                                                     const int32_t *__restrict__ vlist, int32_t *__restrict__ vnext,
                                                     int32_t *pos, const uint16_t *__restrict__ ladj,
                                                     const int2 *__restrict__ range) {
    extern __shared__ uint32_t gp_lds[];
    __shared__ int sh[65];
    __shared__ int32_t ends[2], cut[3], count;
    __shared__ unsigned long long best;
    const int tid = threadIdx.x, nt = blockDim.x;
    const int32_t b = seg[blockIdx.x], k = segk[b], len = k * S, k0 = k / 2, need = k0 * S;
    const int64_t base = (int64_t)b * S;
    const int words = (len + 31) / 32;
    uint32_t *vis = gp_lds;
    uint16_t *dist = reinterpret_cast<uint16_t *>(gp_lds + words), *queue = dist + words * 32;
    if (tid == 0) best = ~0ull;
    __syncthreads();
    for (int i = tid; i < len; i += nt) {
        const int32_t v = vlist[base + i];
        const unsigned long long key = ((unsigned long long)(uint32_t)v << 32) | (uint32_t)i;
        if (key < best) atomicMin(&best, key);
    }
    __syncthreads();
    int level0 = 0, level1 = 0;  // queue range of the last level
    for (int round = 0; round < 2; ++round) {
        const int src = (int)(best & 0xffffffffull);
        __syncthreads();
        for (int i = tid; i < words; i += nt) vis[i] = 0;
        for (int i = tid; i < len; i += nt) dist[i] = 0xffff;
        if (tid == 0) {
            ends[0] = 1;
            cut[0] = -1;  // level at which `need` is reached, its queue range
            best = ~0ull;
        }
        __syncthreads();
        if (tid == 0) {
            vis[src >> 5] = 1u << (src & 31);
            dist[src] = 0;
            queue[0] = (uint16_t)src;
        }
        __syncthreads();
        int head = 0, tail = 1;
        for (int d = 0; head < tail; ++d) {
            level0 = head;
            level1 = tail;
            if (tid == 0 && cut[0] < 0 && tail >= need) {
                cut[0] = d;
                cut[1] = head;
                cut[2] = tail;
            }
            for (int x = head + tid; x < tail; x += nt) {
                const int2 r = range[base + queue[x]];
                for (int32_t q = r.x; q < r.y; q += kNb) {
                    int a[kNb];
#pragma unroll
                    for (int j = 0; j < kNb; ++j) a[j] = ladj[min(q + j, r.y - 1)];
#pragma unroll
                    for (int j = 0; j < kNb; ++j) {
                        const int l = a[j];
                        if (l == 0xffff || (vis[l >> 5] >> (l & 31) & 1)) continue;
                        const uint32_t bit = 1u << (l & 31);
                        if (atomicOr(&vis[l >> 5], bit) & bit) continue;
                        dist[l] = (uint16_t)(d + 1);
                        queue[atomicAdd(&ends[0], 1)] = (uint16_t)l;
                    }
                }
            }
            __syncthreads();
            head = tail;
            tail = ends[0];
            __syncthreads();
        }
        if (round == 0) {  // farthest: smallest vertex of the last level
            for (int x = level0 + tid; x < level1; x += nt) {
                const int i = queue[x];
                const unsigned long long key = ((unsigned long long)(uint32_t)vlist[base + i] << 32) | (uint32_t)i;
                if (key < best) atomicMin(&best, key);
            }
            __syncthreads();
        }
    }
    // vertices nearer than the cut are in; of the cut's distance (the
    // unreached ones if the reached do not suffice) the m of smallest index
    const bool reached = cut[0] >= 0;
    const int dcut = reached ? cut[0] : 0xffff;
    const int c0 = reached ? cut[1] : 0, c1 = reached ? cut[2] : len;
    const int m = need - (reached ? cut[1] : ends[0]);
    uint32_t lo = 0, hi = 0x7fffffffu;  // smallest t with at least m candidates of index <= t
    while (lo < hi) {
        const uint32_t mid = lo + (hi - lo) / 2;
        __syncthreads();
        if (tid == 0) count = 0;
        __syncthreads();
        int c = 0;
        for (int x = c0 + tid; x < c1; x += nt) {
            const int i = reached ? queue[x] : x;
            if (dist[i] == dcut && (uint32_t)vlist[base + i] <= mid) ++c;
        }
#pragma unroll
        for (int j = 32; j >= 1; j >>= 1) c += __shfl_xor(c, j);
        if ((tid & 63) == 0 && c) atomicAdd(&count, c);
        __syncthreads();
        if (count >= m)
            hi = mid;
        else
            lo = mid + 1;
    }
    const uint32_t last = lo;
    int done = 0;
    for (int t0 = 0; t0 < len; t0 += nt) {
        const int i = t0 + tid;
        int32_t v = 0;
        bool in = false;
        if (i < len) {
            v = vlist[base + i];
            in = dist[i] < dcut || (dist[i] == dcut && m > 0 && (uint32_t)v <= last);
        }
        int tot;
        const int before = done + block_excl_scan(in ? 1 : 0, sh, &tot);  // kept vertices before i
        if (i < len) {
            const int at = in ? before : need + (i - before);
            vnext[base + at] = v;
            pos[v] = (int32_t)(base + at);
            if (!in) label[v] = b + k0;
        }
        done += tot;
    }
}

int bits_for(uint64_t x) {
    int b = 0;
    while (b < 64 && (x >> b) != 0) ++b;
    return b < 1 ? 1 : b;
}

}  // namespace

int graph_partition(dd_ctx *h, const int32_t *ptr, const int32_t *col, hipStream_t st) {
    const int64_t n = h->n;
    const int32_t S = h->S, nparts = h->nsub;
    std::vector<void *> tmp;
    auto get = [&](auto **p, int64_t count) -> hipError_t {
        void *q = nullptr;
        hipError_t e = pool_alloc(&q, (size_t)std::max<int64_t>(count, 1) * sizeof(**p));
        if (e == hipSuccess) {
            tmp.push_back(q);
            *p = static_cast<std::remove_reference_t<decltype(*p)>>(q);
        }
        return e;
    };
    auto done = [&](int rc) {
        // kernels may still run after an error; all other exits are synchronised
        const bool idle = hipDeviceSynchronize() == hipSuccess;
        for (void *q : tmp)
            if (idle) pool_free(q); else (void)hipFree(q);
        return rc;
    };
#define GCHK(x)                                                                   \
    do {                                                                          \
        hipError_t e_ = (x);                                                      \
        if (e_ != hipSuccess) {                                                   \
            (void)hipGetLastError();                                              \
            h->fail(DD_EHIP, "graph partition: %s: %s", #x, hipGetErrorString(e_)); \
            return done(DD_EHIP);                                                 \
        }                                                                         \
    } while (0)
    // the last depths split segment by segment; the segments' labels,
    // vertex lists and local adjacency
    int32_t *seg = nullptr, *vlist[2] = {nullptr, nullptr}, *pos = nullptr;
    uint16_t *ladj = nullptr;
    int2 *range = nullptr;
    std::vector<int32_t> segh;
    bool local = false;
    int32_t *label = h->part_id, *segk = nullptr, *src = nullptr, *idx = nullptr, *sorted = nullptr,
            *changed = nullptr;
    uint32_t *dist = nullptr;
    unsigned long long *key = nullptr, *key2 = nullptr, *far = nullptr;
    GCHK(get(&segk, nparts));
    GCHK(get(&src, nparts));
    GCHK(get(&far, nparts));
    GCHK(get(&dist, n));
    GCHK(get(&key, n));
    GCHK(get(&key2, n));
    GCHK(get(&idx, n));
    GCHK(get(&sorted, n));
    GCHK(get(&changed, kLevelBatch));
    size_t temp_bytes = 0, temp32 = 0;
    GCHK(hipcub::DeviceRadixSort::SortPairs(nullptr, temp_bytes, key, key2, idx, sorted, (int)n, 0, 64, st));
    GCHK(hipcub::DeviceRadixSort::SortPairs(nullptr, temp32, reinterpret_cast<uint32_t *>(key),
                                           reinterpret_cast<uint32_t *>(key2), idx, sorted, (int)n, 0, 32, st));
    temp_bytes = std::max(temp_bytes, temp32);
    void *temp = nullptr;
    GCHK(get(reinterpret_cast<unsigned char **>(&temp), (int64_t)temp_bytes));
    const int end_bit = 32 + bits_for((uint64_t)nparts);

    std::vector<int32_t> kh(nparts, 0), next(nparts, 0);
    kh[0] = nparts;
    k_gp_fill<<<blocks(n), kT, 0, st>>>(n, label, 0);
    GCHK(hipGetLastError());

    auto bfs = [&]() -> hipError_t {
        k_gp_src<<<blocks(n), kT, 0, st>>>(n, label, segk, src, dist);
        hipError_t e = hipGetLastError();
        for (uint32_t d = 0; e == hipSuccess && d < (uint32_t)n; d += kLevelBatch) {
            k_gp_fill<<<1, kT, 0, st>>>(kLevelBatch, changed, 0);
            for (int j = 0; j < kLevelBatch; ++j)
                k_gp_level<<<blocks((n + kPer - 1) / kPer), kT, 0, st>>>(n, ptr, col, label, d + j, dist, changed + j);
            int32_t last = 0;
            if ((e = hipGetLastError()) != hipSuccess) break;
            if ((e = hipMemcpyAsync(&last, changed + kLevelBatch - 1, sizeof(int32_t), hipMemcpyDeviceToHost,
                                    st)) != hipSuccess)
                break;
            if ((e = hipStreamSynchronize(st)) != hipSuccess) break;
            if (!last) break;  // no vertex at distance d + kLevelBatch: every segment is exhausted
        }
        return e;
    };

    // part counts of the next depth's segments
    auto halve = [&]() {
        std::fill(next.begin(), next.end(), 0);
        for (int32_t b = 0; b < nparts; ++b) {
            if (kh[b] == 1) next[b] = 1;
            if (kh[b] > 1) {
                next[b] = kh[b] / 2;
                next[b + kh[b] / 2] = kh[b] - kh[b] / 2;
            }
        }
        kh.swap(next);
    };

    for (;;) {
        bool split = false;
        for (int32_t b = 0; b < nparts; ++b) split = split || kh[b] > 1;
        if (!split) break;
        GCHK(hipMemcpyAsync(segk, kh.data(), sizeof(int32_t) * nparts, hipMemcpyHostToDevice, st));
        // Segments that fit one workgroup's LDS take a workgroup each; with
        // parts of more than half that, every depth takes the general way.
        const int32_t kmax = *std::max_element(kh.begin(), kh.end());
        if ((int64_t)kmax * S <= kLocal) {
            if (!local) {
                GCHK(get(&seg, nparts));
                GCHK(get(&pos, n));
                GCHK(get(&vlist[1], n));
                GCHK(get(&ladj, h->nnzb));
                GCHK(get(&range, n));
                GCHK(hipFuncSetAttribute(reinterpret_cast<const void *>(k_gp_local),
                                         hipFuncAttributeMaxDynamicSharedMemorySize, local_lds(kLocal)));
                vlist[0] = sorted;  // the last sort's order holds each new segment as one run
                if (kh[0] == nparts)
                    k_gp_iota<<<blocks(n), kT, 0, st>>>(n, vlist[0], pos);
                else
                    k_gp_pos<<<blocks(n), kT, 0, st>>>(n, vlist[0], pos);
                local = true;
            }
            segh.clear();
            for (int32_t b = 0; b < nparts; ++b)
                if (kh[b] > 1) segh.push_back(b);
            GCHK(hipMemcpyAsync(seg, segh.data(), sizeof(int32_t) * segh.size(), hipMemcpyHostToDevice, st));
            const int per = (int)blocks((int64_t)kmax * S);
            k_gp_adj<<<(unsigned)(segh.size() * per), kT, 0, st>>>(S, per, seg, segk, ptr, col, vlist[0], pos, ladj,
                                                                   range);
            k_gp_local<<<(unsigned)segh.size(), kLocalT, local_lds(kmax * S), st>>>(S, seg, segk, label, vlist[0],
                                                                                  vlist[1], pos, ladj, range);
            GCHK(hipGetLastError());
            GCHK(hipStreamSynchronize(st));  // seg and segk are written again for the next depth
            std::swap(vlist[0], vlist[1]);
            halve();
            continue;
        }
        k_gp_fill<<<blocks(nparts), kT, 0, st>>>(nparts, src, 0x7fffffff);
        const unsigned gx = (unsigned)std::min<int64_t>((n + 1023) / 1024, 512);
        k_gp_extreme<false><<<gx, 1024, 0, st>>>(n, nparts, label, segk, nullptr, src, nullptr);
        GCHK(hipGetLastError());
        GCHK(bfs());
        k_gp_fill64<<<blocks(nparts), kT, 0, st>>>(nparts, far);
        k_gp_extreme<true><<<gx, 1024, 0, st>>>(n, nparts, label, segk, dist, nullptr, far);
        k_gp_far_src<<<blocks(nparts), kT, 0, st>>>(nparts, segk, far, src);
        GCHK(hipGetLastError());
        GCHK(bfs());
        k_gp_keys<<<blocks(n), kT, 0, st>>>(n, label, dist, key, idx);
        GCHK(hipGetLastError());
        GCHK(hipcub::DeviceRadixSort::SortPairs(temp, temp_bytes, key, key2, idx, sorted, (int)n, 0, end_bit, st));
        k_gp_split<<<blocks(n), kT, 0, st>>>(n, S, sorted, segk, label);
        GCHK(hipGetLastError());
        halve();
    }
    // renumber: stable sort of the vertices by label
    uint32_t *lkey = reinterpret_cast<uint32_t *>(key), *lkey2 = reinterpret_cast<uint32_t *>(key2);
    k_gp_label_keys<<<blocks(n), kT, 0, st>>>(n, label, lkey, idx);
    GCHK(hipGetLastError());
    GCHK(hipcub::DeviceRadixSort::SortPairs(temp, temp_bytes, lkey, lkey2, idx, sorted, (int)n, 0,
                                           bits_for((uint64_t)nparts), st));
    k_gp_perm<<<blocks(n), kT, 0, st>>>(n, sorted, h->new2old, h->old2new);
    GCHK(hipGetLastError());
    GCHK(hipStreamSynchronize(st));
#undef GCHK
    return done(DD_OK);
}

}  // namespace ddilu
