// The handle's states on a host without a GPU: the C entry points (api.hip)
// and the memory pool (pool.hip) with the driver and the kernels stood in for.
// Device memory is host memory; a kernel's stand-in checks the buffers it
// would touch and notes which factorisation their contents come from.  Every
// device allocation of a call can be made to fail, and a capture can be in
// progress.
#include <cstdio>
#include <cstdlib>
#include <map>
#include <set>

#include "../paper_2508_04917_amd/csrc/api.hip"
#include "../paper_2508_04917_amd/csrc/pool.hip"

// ---------------------------------------------------------------- driver
static std::set<void *> live;
static long budget = -1;  // device allocations that still succeed (-1: all)
static bool capturing = false, invalidated = false;
static hipStreamCaptureMode mode = hipStreamCaptureModeGlobal;

// a call that a capture in progress does not allow in the present mode
static bool refused() {
    if (!capturing || mode == hipStreamCaptureModeRelaxed) return false;
    invalidated = true;
    return true;
}

hipError_t hipMalloc(void **p, size_t n) {
    if (refused()) return hipErrorStreamCaptureUnsupported;
    if (budget == 0) return hipErrorOutOfMemory;
    if (budget > 0) --budget;
    *p = std::calloc(1, n);
    live.insert(*p);
    return hipSuccess;
}
static std::map<const void *, int> content;  // buffer -> factorisation its contents come from
hipError_t hipFree(void *p) {
    if (refused()) return hipErrorStreamCaptureUnsupported;
    if (live.erase(p) != 1) std::abort();
    content.erase(p);
    std::free(p);
    return hipSuccess;
}
static hipError_t on_stream(hipStream_t st) {
    if (capturing && !st) {
        invalidated = true;
        return hipErrorStreamCaptureImplicit;
    }
    return hipSuccess;
}
hipError_t hipMemcpyAsync(void *d, const void *s, size_t n, hipMemcpyKind, hipStream_t st) {
    std::memcpy(d, s, n);
    return on_stream(st);
}
hipError_t hipMemsetAsync(void *d, int v, size_t n, hipStream_t st) {
    std::memset(d, v, n);
    return on_stream(st);
}
hipError_t hipStreamSynchronize(hipStream_t st) {
    if (refused()) return hipErrorStreamCaptureUnsupported;
    return on_stream(st);
}
hipError_t hipDeviceSynchronize() {
    if (!capturing) return hipSuccess;
    invalidated = true;
    return hipErrorStreamCaptureUnsupported;
}
hipError_t hipStreamCreateWithFlags(hipStream_t *st, unsigned) {
    if (refused()) return hipErrorStreamCaptureUnsupported;
    *st = reinterpret_cast<hipStream_t>(std::malloc(1));
    return hipSuccess;
}
hipError_t hipStreamDestroy(hipStream_t st) {
    std::free(st);
    return hipSuccess;
}
hipError_t hipThreadExchangeStreamCaptureMode(hipStreamCaptureMode *m) {
    std::swap(*m, mode);
    return hipSuccess;
}
hipError_t hipGetDevice(int *d) {
    *d = 0;
    return hipSuccess;
}
hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipGetLastError() { return hipSuccess; }
hipError_t hipMemGetInfo(size_t *f, size_t *t) {
    *f = *t = size_t(16) << 30;
    return hipSuccess;
}
hipError_t hipDeviceGetAttribute(int *v, hipDeviceAttribute_t, int) {
    *v = 163840;
    return hipSuccess;
}
const char *hipGetErrorString(hipError_t) { return "error"; }
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
hipError_t hipHostFree(void *) { return hipSuccess; }

// --------------------------------------------------------------- kernels
enum Layout { DIRECT, SLOTS, SEGMENTED, CSR };
static Layout layout = DIRECT;
static bool singular = false;
static int factorisation = 0;
static int wrong = 0;  // a kernel would have read or written through a null or stale pointer

static void need(const void *p, const char *what) {
    if (p && live.count(const_cast<void *>(p))) return;
    std::printf("  missing buffer: %s\n", what);
    ++wrong;
}
static void put(const void *p, const char *what) {
    need(p, what);
    if (p) content[p] = factorisation;
}
static void get(const void *p, const char *what) {
    need(p, what);
    if (p && content[p] != factorisation) {
        std::printf("  stale contents: %s\n", what);
        ++wrong;
    }
}

namespace ddilu {
int64_t scan_tmp_elems(int64_t) { return 2; }
hipError_t exclusive_scan(const int32_t *in, int32_t *out, int64_t n, int32_t *, hipStream_t st) {
    int32_t s = 0;
    for (int64_t i = 0; i < n; ++i) {
        const int32_t v = in[i];
        out[i] = s;
        s += v;
    }
    out[n] = s;
    return on_stream(st);
}
hipError_t launch_check_rows(int64_t, int64_t, const int32_t *, const int32_t *, int32_t *, hipStream_t) { return hipSuccess; }
hipError_t launch_partition(dd_ctx *, hipStream_t) { return hipSuccess; }
int graph_partition(dd_ctx *, const int32_t *, const int32_t *, hipStream_t) { return DD_OK; }
hipError_t launch_row_len(dd_ctx *h, const int32_t *ptr, int32_t *len, hipStream_t) {
    for (int64_t i = 0; i < h->n; ++i) len[i] = ptr[i + 1] - ptr[i];
    return hipSuccess;
}
hipError_t launch_reorder_rows(dd_ctx *, const int32_t *, const int32_t *, int32_t *, hipStream_t) { return hipSuccess; }
void build_spmv_layout(dd_ctx *, hipStream_t) {}
hipError_t launch_values(dd_ctx *h, const double *, const int32_t *, hipStream_t st) {
    need(h->aval, "aval");
    return on_stream(st);
}
hipError_t launch_gather_blocks(int64_t, int, const int32_t *src, const double *, double *out, hipStream_t st) {
    need(src, "gather source");
    need(out, "gathered blocks");
    return on_stream(st);
}
hipError_t launch_drop_count(dd_ctx *h, int32_t *, int32_t *tlen, hipStream_t) {
    for (int64_t i = 0; i < h->n; ++i) tlen[i] = h->aptr[i + 1] - h->aptr[i];
    return hipSuccess;
}
hipError_t launch_drop_rows(dd_ctx *h, const int32_t *tbeg, int32_t *tsrc, hipStream_t) {
    need(tbeg, "tbeg");
    need(tsrc, "tsrc");
    need(h->tcol, "tcol");
    need(h->tdiag, "tdiag");
    return hipSuccess;
}
hipError_t launch_level_sets(dd_ctx *h, int32_t *stats, hipStream_t) {
    const int most = layout == CSR ? 60 : layout == SEGMENTED ? 10 : 3;
    stats[0] = stats[1] = most;
    stats[2] = stats[3] = 2;
    stats[6] = stats[7] = (int32_t)h->nnzt;
    for (int w = 0; w < 2; ++w)
        for (int s = 0; s < h->nsub; ++s) h->lev[w].nlev[s] = 2;
    return hipSuccess;
}
hipError_t launch_plus_one(int64_t m, const int32_t *in, int32_t *out, hipStream_t) {
    for (int64_t i = 0; i < m; ++i) out[i] = in[i] + 1;
    return hipSuccess;
}
hipError_t launch_level_lists(dd_ctx *h, int32_t *stats, hipStream_t) {
    stats[4] = 4;
    for (int w = 0; w < 2; ++w) need(h->lev[w].ptr, "level lists");
    return hipSuccess;
}
int build_wave_chunks(dd_ctx *h, int which, hipStream_t) {
    Sweep &w = h->sw[which];
    h->release(w.wtab);
    h->release(w.winfo);
    int rc = h->alloc(&w.wtab, w.snpos);
    if (!rc) rc = h->alloc(&w.winfo, h->nsub);
    return rc;
}
hipError_t launch_slot_records(dd_ctx *h, int32_t *stats, hipStream_t) {
    stats[0] = layout == SLOTS;
    need(h->frec, "frec");
    for (int w = 0; w < 2; ++w) need(h->sw[w].desc, "desc");
    return hipSuccess;
}
static void factored(dd_ctx *h) {
    ++factorisation;
    if (singular) h->status[2] = 0;
    put(h->invd, "invd");
}
hipError_t launch_bilu0(dd_ctx *h, hipStream_t) {
    factored(h);
    put(h->lu, "lu");
    return hipSuccess;
}
hipError_t launch_bilu0_slots(dd_ctx *h, hipStream_t) {
    factored(h);
    for (int w = 0; w < 2; ++w) {
        need(h->sw[w].desc, "desc");
        put(h->sw[w].sval64, "sval64");
    }
    return hipSuccess;
}
hipError_t launch_lu_blocks(dd_ctx *h, hipStream_t st) {
    if (!h->direct) return hipSuccess;
    get(h->sw[0].sval64, "sval64");
    put(h->lu, "lu");
    return on_stream(st);
}
hipError_t launch_export_factors(dd_ctx *, double *, hipStream_t) { return hipSuccess; }
hipError_t launch_pack_count(dd_ctx *h, int which, int32_t *cnt, hipStream_t st) {
    need(cnt, "counts");
    need(h->sw[which].prow, "prow");
    for (int64_t i = 0; i < h->n; ++i) cnt[i] = 1;
    return on_stream(st);
}
hipError_t launch_pack_fill(dd_ctx *h, int which, hipStream_t st) {
    Sweep &s = h->sw[which];
    get(h->lu, "lu");
    need(s.bptr, "bptr");
    need(s.bcol, "bcol");
    put(s.val64, "val64");
    if (which) put(s.d64, "d64");
    return on_stream(st);
}
hipError_t launch_pack_unscaled(dd_ctx *h, hipStream_t) {
    get(h->lu, "lu");
    put(h->sw[1].uraw, "uraw");
    return hipSuccess;
}
hipError_t launch_pack_slots(dd_ctx *h, int which, hipStream_t) {
    get(h->lu, "lu");
    put(h->sw[which].sval64, "sval64");
    return hipSuccess;
}
hipError_t launch_seg_pack(dd_ctx *h, hipStream_t) {
    get(h->lu, "lu");
    for (int w = 0; w < 2; ++w) {
        need(h->sw[w].desc, "desc");
        put(h->sw[w].sval64, "sval64");
    }
    return hipSuccess;
}
int build_seg_layout(dd_ctx *h, hipStream_t st) {
    for (int w = 0; w < 2; ++w) {
        Sweep &s = h->sw[w];
        h->release(s.pmap);
        h->release(s.wtab);
        h->release(s.winfo);
        s.snpos = 2 * h->n;
        int rc = h->alloc(&s.pmap, s.snpos);
        if (!rc) rc = h->alloc(&s.wtab, s.snpos);
        if (!rc) rc = h->alloc(&s.winfo, h->nsub);
        if (!rc) rc = h->alloc(&s.desc, s.snpos);
        if (!rc) rc = h->alloc(&s.sval64, s.snpos);
        if (rc) return rc;
    }
    return launch_seg_pack(h, st) == hipSuccess ? DD_OK : DD_EHIP;
}
hipError_t launch_cast32(dd_ctx *h, hipStream_t st) {  // as the real one: what is there, and both slot streams
    for (int w = 0; w < 2; ++w)
        if (h->sw[w].val32) {
            get(h->sw[w].val64, "val64");
            put(h->sw[w].val32, "val32");
        }
    if (h->csr_ready && h->sw[1].d32) {
        get(h->sw[1].d64, "d64");
        put(h->sw[1].d32, "d32");
    }
    if (h->slots || h->seg)
        for (int w = 0; w < 2; ++w) {
            get(h->sw[w].sval64, "sval64");
            put(h->sw[w].sval32, "sval32");
        }
    return on_stream(st);
}
// the route of the real launch and the buffers its kernel reads
static hipError_t route(dd_ctx *h, int precision) {
    const bool fp32 = precision != DD_FP64;
    if ((h->variant == 0 || h->variant == 3) && (h->slots || h->seg)) {
        for (int w = 0; w < 2; ++w) {
            need(h->sw[w].desc, "desc");
            need(h->sw[w].wtab, "wtab");
            need(h->sw[w].winfo, "winfo");
            if (fp32)
                get(h->sw[w].sval32, "sval32");
            else
                get(h->sw[w].sval64, "sval64");
        }
        return hipSuccess;
    }
    if (!h->csr_ready) return hipErrorInvalidValue;
    if (fp32 && (!h->sw[0].val32 || !h->sw[1].val32 || !h->sw[1].d32)) return hipErrorInvalidValue;
    for (int w = 0; w < 2; ++w) {
        need(h->sw[w].bcol, "bcol");
        if (fp32)
            get(h->sw[w].val32, "val32");
        else
            get(h->sw[w].val64, "val64");
    }
    if (fp32)
        get(h->sw[1].d32, "d32");
    else
        get(h->sw[1].d64, "d64");
    if (h->variant == 7) get(h->sw[1].uraw, "uraw");
    return hipSuccess;
}
hipError_t launch_apply(dd_ctx *h, const double *, double *, const int32_t *, hipStream_t) { return route(h, h->precision); }
const char *variant_unsupported(const dd_ctx *h, int v) {
    return v >= 4 && h->precision != DD_FP64 ? "precision" : nullptr;
}
int apply_lds_bytes(const dd_ctx *, int) { return 0; }
// a training step applies whether or not the handle is factored
int lic_loss_grad_run(dd_ctx *h, const float *, int, const double *, const double *, const double *, double *, float *, int,
                      hipStream_t) {
    return route(h, DD_FP64) == hipSuccess ? DD_OK : DD_EHIP;
}
int lic_setup(dd_ctx *, hipStream_t) { return DD_OK; }
int lic_publish_coeffs(dd_ctx *, hipStream_t) { return DD_OK; }
int lic_coeffs_from_params(dd_ctx *, const float *, bool, hipStream_t) { return DD_OK; }
int lic_adjoint_streams(dd_ctx *, hipStream_t) { return DD_OK; }
int lic_targets_run(dd_ctx *, int, const double *, double *, double *, hipStream_t) { return DD_OK; }
int bicgstab_run(dd_ctx *, const KrylovWork &, const double *, double *, double, int, hipStream_t, dd_solve_info *) { return DD_OK; }
int krylov_workspace(dd_ctx *, KrylovWork *) { return DD_OK; }
int noalloc_workspace(dd_ctx *, KrylovWork *, KrylovScalars *) { return DD_OK; }
int global_factor(dd_ctx *, hipStream_t) { return DD_OK; }
hipError_t launch_global_apply(dd_ctx *, const double *, double *, int, hipStream_t) { return hipSuccess; }
hipError_t launch_apply_adjoint(dd_ctx *, const double *, double *, int, hipStream_t) { return hipSuccess; }
hipError_t launch_spmv(dd_ctx *, const double *, double *, hipStream_t) { return hipSuccess; }
hipError_t launch_adam(int, float *, const float *, float *, float *, int, float, float, float, float, hipStream_t) { return hipSuccess; }
}  // namespace ddilu

// ----------------------------------------------------------------- tests
static int errors = 0;
#define CHECK(c)                                                        \
    do {                                                                \
        if (!(c)) {                                                     \
            std::printf("line %d: %s\n", __LINE__, #c);                 \
            ++errors;                                                   \
        }                                                               \
    } while (0)

constexpr int N = 32, PART = 8, PER = 3;
static double vec[2][N * 9], values[N * PER * 9];

static dd_handle partition() {
    static int32_t ptr[N + 1], col[N * PER];
    for (int i = 0; i <= N; ++i) ptr[i] = PER * i;
    dd_graph_desc d{};
    d.n = N;
    d.bs = 3;
    d.part_rows = PART;
    d.lds_budget_bytes = 163840;
    d.n_cu = 256;
    dd_handle h = nullptr;
    CHECK(dd_partition_graph(&d, ptr, col, values, N * PER, nullptr, &h) == DD_OK);
    return h;
}

static int apply(dd_handle h) { return dd_trsv_apply(h, vec[0], vec[1], nullptr); }
static int train(dd_handle h) {  // refused unless the handle's faces are set up
    return lic_loss_grad(h, (float *)vec[0], 1, vec[0], vec[0], vec[0], vec[1], (float *)vec[1], 0, nullptr);
}

// what every handle may do whatever happened before: succeed or refuse
static void poke(dd_handle h) {
    (void)apply(h);
    (void)train(h);
}

// `call` with every device allocation it makes failing in turn, each time on
// the state the failure before left; then without failures
template <typename F>
static void robust(dd_handle h, const char *what, F call) {
    for (long k = 0;; ++k) {
        ddilu::pool_trim(-1);
        const int before = wrong;
        budget = k;
        const int rc = call();
        budget = -1;
        if (!h->retired.empty()) {
            std::printf("layout %d, %s, allocation %ld: %zu buffers not given back\n", layout, what, k, h->retired.size());
            ++errors;
            return;
        }
        if (rc != DD_OK) {
            CHECK(rc == DD_ENOMEM);
            poke(h);
        }
        if (wrong != before) {
            std::printf("layout %d, %s, allocation %ld\n", layout, what, k);
            return;
        }
        if (rc == DD_OK) break;
        if (k > 200) {
            std::printf("layout %d, %s never succeeds\n", layout, what);
            ++errors;
            return;
        }
    }
}

static void applies(dd_handle h) {
    for (int v : {0, 1, 2, 3, 4, 7, 0}) {
        robust(h, "dd_set_apply_variant", [&] {
            const int was = h->variant, rc = dd_set_apply_variant(h, v);
            CHECK(rc == DD_OK || h->variant == was);
            return rc;
        });
        for (int p : {DD_MIXED, DD_FP64, DD_FP32, DD_FP64}) {
            robust(h, "dd_set_precision", [&] { return dd_set_precision(h, p, nullptr); });
            if (v >= 4 && p != DD_FP64) continue;
            robust(h, "dd_trsv_apply", [&] { return apply(h); });
        }
    }
}

static void states(Layout l) {
    layout = l;
    dd_handle h = partition();
    for (int precision : {DD_MIXED, DD_FP64}) {
        robust(h, "ilu0_factor", [&] { return ilu0_factor(h, precision, nullptr); });
        CHECK(apply(h) == DD_OK);
        h->lic.ready = 1;  // lic_setup, until the next refactorisation
        applies(h);
        robust(h, "ilu0_factor of a factored handle", [&] { return ilu0_factor(h, precision, nullptr); });
        CHECK(apply(h) == DD_OK && train(h) == DD_OK);
        robust(h, "ilu0_refactor", [&] { return ilu0_refactor(h, values, nullptr); });
        applies(h);
        // a variant chosen while the handle is not factored
        for (int v : {1, 2, 7, 0}) {
            if (v == 7 && precision != DD_FP64) continue;
            CHECK(dd_set_apply_variant(h, 0) == DD_OK);
            robust(h, "ilu0_factor again", [&] { return ilu0_factor(h, precision, nullptr); });
            singular = true;
            CHECK(ilu0_refactor(h, values, nullptr) == DD_EZEROPIVOT);
            singular = false;
            poke(h);
            CHECK(apply(h) == DD_ESTATE);
            CHECK(dd_set_apply_variant(h, v) == DD_OK);
            robust(h, "ilu0_refactor after a failure", [&] { return ilu0_refactor(h, values, nullptr); });
            CHECK(apply(h) == DD_OK);
        }
        singular = true;
        CHECK(ilu0_factor(h, precision, nullptr) == DD_EZEROPIVOT);
        singular = false;
        poke(h);
        CHECK(apply(h) == DD_ESTATE);
        CHECK(ilu0_refactor(h, values, nullptr) == DD_ESTATE);
    }
    dd_destroy(h);
    dd_destroy(nullptr);
    CHECK(live.empty());
}

static void during_capture(Layout l, int precision) {
    layout = l;
    dd_handle h = partition();
    CHECK(ilu0_factor(h, precision, nullptr) == DD_OK);
    capturing = true;
    CHECK(dd_set_apply_variant(h, 1) == DD_OK);
    CHECK(dd_set_apply_variant(h, 0) == DD_OK);
    capturing = false;
    CHECK(!invalidated && mode == hipStreamCaptureModeGlobal);
    invalidated = false;
    CHECK(dd_set_apply_variant(h, 1) == DD_OK && apply(h) == DD_OK);
    dd_destroy(h);
    dd_destroy(nullptr);
    CHECK(live.empty());
}

int main() {
    for (Layout l : {DIRECT, SLOTS, SEGMENTED, CSR}) {
        states(l);
        during_capture(l, DD_FP64);
        during_capture(l, DD_MIXED);
    }
    std::printf("%d wrong accesses, %d errors\n", wrong, errors);
    return wrong || errors;
}
