// host_checks.cpp -- checks of the library's host code without a GPU: the
// host sources (cgmi.cpp, devmatrix.cpp, staged.cpp, fsai.cpp) are linked with
// the HIP calls below, which keep "device" memory on the host, and with
// kernel launches that record what they are asked for or do nothing (those
// that no check reaches stay unresolved).
//
//     host_checks staged ROWS COLS PER_ROW
//         the staged column segments of a matrix of ROWS rows, PER_ROW random
//         entries each (every fifth row twice as many, one row 1500), all
//         columns below COLS: every index the product's kernel forms lies in
//         its buffer, and the sums are the rows' own.  Says whether the
//         schedule runs its products on them
//     host_checks widths
//         the widths of segments for numbers of columns and widest segments
//     host_checks mixed
//         a handle turned to mixed precision keeps no staged column segments,
//         and has the same ones when it is turned back
//     host_checks stage
//         a trainer's steps after a page-locked allocation failed: none writes
//         past the buffer that a later one got
//     host_checks abandoned
//         a solve in one launch whose workgroups did not all run at once is
//         made with the separate kernels
//     host_checks streams
//         products and a solve through one handle on several streams: where
//         they share the staged sums, each runs after the one before
#include <hip/hip_runtime_api.h>

#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <random>
#include <string>
#include <vector>

#include "../../include/cgmi_fsai.h"
#include "../../paper_2608_09647_amd/csrc/cgmi_host.h"
#include "../../paper_2608_09647_amd/csrc/fsai_internal.h"

using namespace cgmi;

// ---------------------------------------------------------------------------
// HIP on host memory

extern "C" {
hipError_t hipMalloc(void **p, size_t n) { return (*p = std::malloc(n)) ? hipSuccess : hipErrorOutOfMemory; }
hipError_t hipFree(void *p) {
    std::free(p);
    return hipSuccess;
}
hipError_t hipMemcpy(void *d, const void *s, size_t n, hipMemcpyKind) {
    std::memcpy(d, s, n);
    return hipSuccess;
}
hipError_t hipMemset(void *d, int v, size_t n) {
    std::memset(d, v, n);
    return hipSuccess;
}
hipError_t hipMemcpyAsync(void *d, const void *s, size_t n, hipMemcpyKind k, hipStream_t) { return hipMemcpy(d, s, n, k); }
hipError_t hipMemsetAsync(void *d, int v, size_t n, hipStream_t) { return hipMemset(d, v, n); }
// Page-locked memory: its size in front, kGuard bytes behind that nothing writes.
constexpr size_t kHead = 64, kGuard = 1 << 16;
static bool g_no_pinned = false, g_overrun = false;
hipError_t hipHostMalloc(void **p, size_t n, unsigned) {
    if (g_no_pinned) return hipErrorOutOfMemory;
    unsigned char *const b = static_cast<unsigned char *>(std::malloc(kHead + n + kGuard));
    std::memcpy(b, &n, sizeof n);
    std::memset(b + kHead + n, 0xA5, kGuard);
    *p = b + kHead;
    return hipSuccess;
}
hipError_t hipHostFree(void *p) {
    if (!p) return hipSuccess;
    unsigned char *const b = static_cast<unsigned char *>(p) - kHead;
    size_t n;
    std::memcpy(&n, b, sizeof n);
    for (size_t i = 0; i < kGuard; ++i) g_overrun |= b[kHead + n + i] != 0xA5;
    std::free(b);
    return hipSuccess;
}
hipError_t hipGetDeviceCount(int *n) { return *n = 1, hipSuccess; }
hipError_t hipGetDevice(int *d) { return *d = 0, hipSuccess; }
hipError_t hipDeviceGetAttribute(int *v, hipDeviceAttribute_t, int) { return *v = 100000, hipSuccess; }
hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipGetLastError() { return hipSuccess; }
const char *hipGetErrorString(hipError_t) { return "error"; }
}

// Streams and events by what is known to have ended before the next command
// on a stream: the number of the last product.
struct ihipStream_t {
    bool capture = false;
    int after = 0;
};
struct ihipEvent_t {
    int after = 0;
};
static int g_products = 0, g_ended = 0, g_waits = 0, g_events = 0;
static std::string g_fault;

extern "C" {
hipError_t hipEventCreateWithFlags(hipEvent_t *e, unsigned) {
    ++g_events;
    return *e = new ihipEvent_t(), hipSuccess;
}
hipError_t hipEventDestroy(hipEvent_t e) {
    delete e;
    return hipSuccess;
}
hipError_t hipEventRecord(hipEvent_t e, hipStream_t s) {
    if (s->capture) g_fault = "an event recorded under capture";
    e->after = s->after;
    return hipSuccess;
}
hipError_t hipStreamWaitEvent(hipStream_t s, hipEvent_t e, unsigned) {
    if (s->capture) g_fault = "a wait under capture";
    s->after = std::max(s->after, e->after);
    ++g_waits;
    return hipSuccess;
}
hipError_t hipDeviceSynchronize() {
    g_ended = g_products;
    ++g_waits;
    return hipSuccess;
}
hipError_t hipStreamIsCapturing(hipStream_t s, hipStreamCaptureStatus *status) {
    *status = s->capture ? hipStreamCaptureStatusActive : hipStreamCaptureStatusNone;
    return hipSuccess;
}
hipError_t hipStreamSynchronize(hipStream_t s) {
    if (s) g_ended = std::max(g_ended, s->after);
    return hipSuccess;
}
}

namespace cgmi {
hipError_t staged_setup() { return hipSuccess; }
static std::vector<unsigned char> g_scratch(kScratchBytes);
hipError_t scratch_setup() { return hipSuccess; }
hipError_t scratch_region(int, void **p, size_t *n) { return *p = g_scratch.data(), *n = g_scratch.size(), hipSuccess; }
hipError_t launch_state_init(DevState *st, double tol, int32_t maxit, double, hipStream_t) {
    *st = DevState{};
    st->tol = tol;
    st->maxit = maxit;
    return hipSuccess;
}
int device_cu_count() { return 256; }
int small_path_max_rows() { return 4096; }
// One launch, which is abandoned: the state keeps saying that it runs.
static bool g_one_launch = false;
static int g_launches = 0;
int resident_groups(int32_t, int32_t, int) { return g_one_launch ? 8 : 0; }
hipError_t launch_cg_resident(const ResidentArgs &a, int32_t, int, hipStream_t) {
    ++g_launches;
    a.st->done = kDoneRunning;
    return hipSuccess;
}
// Ends a solve at once: the state copied back says so (all memory is the host's).
hipError_t launch_spmv(const CsrDev &A, const Schedule &, int, const double *, double *, const double *, const double *,
                       double *, double *, Partials, Partials, DevState *st, int, int, hipStream_t s) {
    if (A.st64 && s && !s->capture) {
        if (std::max(s->after, g_ended) < g_products) g_fault = "a product beside one that is not known to have ended";
        s->after = ++g_products;
    }
    if (st) st->done = kDoneConverged;
    return hipSuccess;
}
hipError_t launch_update_r(int32_t, int, double *, const double *, double *, Partials, DevState *, int, hipStream_t) {
    return hipSuccess;
}
hipError_t launch_update_pxb(int32_t, int, double *, const double *, const double *, double *, Partials, DevState *, int,
                             hipStream_t) {
    return hipSuccess;
}
hipError_t fsai_prepare(int32_t, const int32_t *, const int32_t *, const double *, int32_t *, float *, double *,
                        uint16_t *, int32_t *, hipStream_t) {
    return hipSuccess;
}
hipError_t fsai_forward_outputs(int32_t, const int32_t *, int64_t, const uint16_t *, const float *, float *, int64_t *,
                                hipStream_t) {
    return hipSuccess;
}
hipError_t fsai_loss(int32_t, int32_t, const int32_t *, const int64_t *, const int32_t *, const float *,
                     const int32_t *, const float *, int64_t *, float, double *, hipStream_t) {
    return hipSuccess;
}
hipError_t fsai_backward(int32_t, const int32_t *, const uint16_t *, const float *, const float *, const int64_t *,
                         const int32_t *, float *, int32_t, hipStream_t) {
    return hipSuccess;
}
hipError_t fsai_adam(int32_t, const double *, double *loss, int32_t, const float *, float *, float *, float *, float *,
                     int32_t, float, hipStream_t) {
    *loss = 0.0;
    return hipSuccess;
}
bool spmv_dir_applies(const CsrDev &, const Schedule &, int, const void *, const void *, const void *, const void *,
                      const void *) {
    return false;
}
}  // namespace cgmi

// ---------------------------------------------------------------------------

namespace {

[[noreturn]] void die(const std::string &what) {
    std::printf("FAILED: %s\n", what.c_str());
    std::exit(1);
}
#define REQUIRE(cond, ...)                                   \
    do {                                                     \
        if (!(cond)) {                                       \
            char text_[256];                                 \
            std::snprintf(text_, sizeof text_, __VA_ARGS__); \
            die(std::string(#cond) + ": " + text_);          \
        }                                                    \
    } while (0)

// per_row entries a row, in every fifth row twice as many, in one 1500 (which
// keeps the schedule from stream tiles), one in each of as many equal ranges of
// the columns, integer values (their sums are exact in any order); the last
// column is used.
struct Matrix {
    std::vector<int32_t> rp, ci;
    std::vector<double> val;
};
Matrix random_rows(int32_t rows, int32_t cols, int32_t per_row) {
    Matrix A;
    std::mt19937 rng(7);
    A.rp.assign(1, 0);
    for (int32_t i = 0; i < rows; ++i) {
        const int32_t len = i == rows / 2 ? 1500 : i % 5 ? per_row : 2 * per_row, width = cols / len;
        REQUIRE(width > 0, "%d columns for %d entries a row", cols, len);
        for (int32_t j = 0; j < len; ++j) {
            A.ci.push_back(j * width + (int32_t)(rng() % (uint32_t)width));
            A.val.push_back((double)(int32_t)(rng() % 17u) - 8.0);
        }
        A.rp.push_back((int32_t)A.ci.size());
    }
    A.ci.back() = cols - 1;
    return A;
}

// The product of the staged layout S, entry by entry with the indices the
// kernel forms: list bounds, entry loads (those ahead too), the pieces of p
// staged for every thread, columns and slots in LDS.
std::vector<double> staged_product(const StagedDev &S, const std::vector<double> &p, size_t entries) {
    constexpr int threads = kStagedWaves * kWaveSize, E = 16 / (int)sizeof(double);
    const int chunks = (S.seg_cols * (int)sizeof(double) / 16 + threads - 1) / threads <= 3 ? 3 : 4;
    REQUIRE(S.nseg >= 2 && S.seg_cols % 256 == 0 && S.seg_cols * (int)sizeof(double) <= 16 * threads * kStagedChunks,
            "%d segments of %d", S.nseg, S.seg_cols);
    REQUIRE(staged_lds(S.seg_cols, S.max_slots) <= kStagedLds, "%d columns, %d slots", S.seg_cols, S.max_slots);
    REQUIRE((int64_t)(S.nseg - 1) * S.seg_cols < S.ncols && (int64_t)S.nseg * S.seg_cols >= S.ncols,
            "%d segments of %d for %d columns", S.nseg, S.seg_cols, S.ncols);
    // what segment_load reads, and what segment_store leaves in LDS
    std::vector<std::vector<double>> lds((size_t)S.nseg, std::vector<double>((size_t)S.seg_cols, NAN));
    for (int32_t seg = 0; seg < S.nseg + 2; ++seg) {
        const int32_t s = std::min(seg, S.nseg - 1);
        const int64_t first = (int64_t)s * S.seg_cols;
        for (int32_t u = 0; u < chunks; ++u)
            for (int32_t t = 0; t < threads; ++t) {
                const int32_t k = (u * threads + t) * E;
                int64_t at = first + k;
                if (!(seg < S.nseg - 1 && S.seg_cols == chunks * threads * E)) {
                    const int32_t last = staged_last_pair(S.ncols - s * S.seg_cols, S.seg_cols);
                    at = first + (int64_t)(uint32_t)std::min(k, last);
                }
                REQUIRE(at >= 0 && at + E <= S.ncols, "segment %d of %d reads p[%lld] of %d", (int)seg, S.nseg,
                        (long long)at, S.ncols);
                if (seg < S.nseg && k < S.seg_cols)
                    for (int e = 0; e < E; ++e) lds[(size_t)seg][(size_t)(k + e)] = p[(size_t)(at + e)];
            }
        if (seg == S.nseg - 1)
            for (int32_t c = S.ncols / E * E; c < S.ncols; ++c) {
                REQUIRE(c - first >= 0 && c - first < S.seg_cols, "tail column %d of segment %d", c, seg);
                lds[(size_t)seg][(size_t)(c - first)] = p[(size_t)c];
            }
    }
    const size_t lists = (size_t)S.nblocks * kStagedWaves * S.nseg;
    REQUIRE(S.off[0] == 0 && (size_t)S.off[lists] <= entries, "%d entries", S.off[lists]);
    std::vector<double> q((size_t)S.m, 0.0);
    for (int32_t b = 0; b < S.nblocks; ++b)
        for (int32_t g = 0; g < S.ngroups; ++g) {
            std::vector<double> y((size_t)S.nslots[b] + 1, 0.0);
            REQUIRE(S.nslots[b] <= S.max_slots, "block %d", b);
            const int32_t first = (int32_t)((int64_t)S.nseg * g / S.ngroups);
            const int32_t last = (int32_t)((int64_t)S.nseg * (g + 1) / S.ngroups);
            REQUIRE(first < last, "group %d of %d has no segment (of %d)", g, S.ngroups, S.nseg);
            for (int w = 0; w < kStagedWaves; ++w)
                for (int32_t s = first; s < last; ++s) {
                    const size_t l = ((size_t)b * kStagedWaves + w) * S.nseg + s;
                    const int32_t beg = S.off[l], end = S.off[l + 1];
                    REQUIRE(beg >= 0 && beg <= end && (size_t)beg + kStagedSlack <= entries, "list %zu", l);
                    for (int32_t k = beg; k < end; ++k) {
                        const uint32_t col = staged_col(S.idx[k]), slot = staged_slot(S.idx[k]);
                        REQUIRE((int)slot <= S.nslots[b], "slot %u of %d", slot, S.nslots[b]);
                        REQUIRE((int)col < S.seg_cols, "column %u", col);
                        if ((int)slot < S.nslots[b]) y[slot] += S.val[k] * lds[(size_t)s][col];
                    }
                }
            for (int32_t r = S.row0[(size_t)b * kStagedWaves]; r < S.row0[((size_t)b + 1) * kStagedWaves]; ++r) {
                const uint32_t u = S.slots ? S.slots[r] : (uint32_t)(r - S.row0[(size_t)b * kStagedWaves]) | 1u << 16;
                for (uint32_t i = 0; i < u >> 16; ++i) q[(size_t)r] += y[(u & 0xFFFFu) + i];
            }
        }
    return q;
}

void check_staged(int32_t rows, int32_t cols, int32_t per_row) {
    const int cus = 256;
    const Matrix A = random_rows(rows, cols, per_row);
    DevMatrix M;
    REQUIRE(dm_upload(M, rows, A.rp.data(), A.ci.data(), A.val.data(), 0) == CG_OK, "upload");
    REQUIRE(dm_schedule(M, 0, 0, cus, 16 * cus, false) == CG_OK, "schedule");
    std::printf("%s ", M.use_st64 ? "taken" : "not taken");
    if (M.st64.state == 0) staged_build(M, cus, M.st64);
    if (M.st64.state < 0) {
        std::printf("not built\n");
        dm_free(M);
        return;
    }
    const StagedDev &S = M.st64.dev;
    std::printf("groups %d segments %d of %d columns, %d in the last\n", S.ngroups, S.nseg, S.seg_cols,
                S.ncols - (S.nseg - 1) * S.seg_cols);
    REQUIRE(S.ncols == cols && S.m == rows, "%d x %d", S.m, S.ncols);
    std::vector<double> p((size_t)cols);
    std::mt19937 rng(9);
    for (double &v : p) v = (double)(int32_t)(rng() % 17u) - 8.0;
    const std::vector<double> q = staged_product(S, p, (size_t)(M.nnz + M.nnz / 8) + kStagedSlack);
    for (int32_t i = 0; i < rows; ++i) {
        double s = 0.0;
        for (int32_t k = A.rp[(size_t)i]; k < A.rp[(size_t)i + 1]; ++k)
            s += A.val[(size_t)k] * p[(size_t)A.ci[(size_t)k]];
        REQUIRE(s == q[(size_t)i], "row %d: %g, not %g", i, q[(size_t)i], s);
    }
    dm_free(M);
}

// Every remainder of the last segment but one column, none of them empty; the
// equal parts as long as their last one is no single column.
void check_widths() {
    std::mt19937 rng(3);
    for (int32_t widest = 256; widest <= 8192; widest += 256)
        for (int32_t k = 0; k < 20000; ++k) {
            // whole segments and up to 3 columns more, and any number
            const int32_t n = k & 1 ? widest * (2 + k / 8) + (k / 2) % 4 : 16384 + (int32_t)(rng() % 4000000u);
            const int32_t w = staged_width(n, widest + (int32_t)(rng() % 256u));
            if (w == 0) continue;
            const int32_t nseg = (n + w - 1) / w, left = n - (nseg - 1) * w;
            REQUIRE(w % 256 == 0 && w > 0 && w <= widest, "%d columns, at most %d: %d", n, widest, w);
            REQUIRE(left >= 2 && left <= w, "%d columns by %d: %d left", n, w, left);
        }
    REQUIRE(staged_width(299521, 7771) == 7424 && staged_width(299522, 7771) == 7680, "299521 and 299522 columns");
}

void check_mixed() {
    const int32_t n = 200003;
    const Matrix A = random_rows(n, n, 33);
    DevMatrix M;
    REQUIRE(dm_upload(M, n, A.rp.data(), A.ci.data(), A.val.data(), 0) == CG_OK, "upload");
    auto schedule = [&](bool mixed) { REQUIRE(dm_schedule(M, 0, 0, 256, 4096, mixed) == CG_OK, "schedule"); };
    schedule(false);
    REQUIRE(M.use_st64, "no staged segments");
    const size_t lists = (size_t)M.st64.dev.nblocks * kStagedWaves * M.st64.dev.nseg;
    const std::vector<int32_t> off(M.st64.dev.off, M.st64.dev.off + lists + 1);
    const std::vector<uint32_t> idx(M.st64.dev.idx, M.st64.dev.idx + off[lists]);
    schedule(true);
    REQUIRE(!M.use_st64 && !M.st64.dev.idx && !M.st64.dev.part, "still held");
    schedule(false);
    REQUIRE(M.use_st64 && std::equal(off.begin(), off.end(), M.st64.dev.off) &&
                std::equal(idx.begin(), idx.end(), M.st64.dev.idx), "another layout");
    dm_free(M);
}

void check_stage() {
    constexpr int32_t nsys = 4, n = 64;
    std::vector<int32_t> rp(n + 1), ci(n), sizes(nsys, n), sys{0, 1, 2, 3}, rows(4 * 1024, 1);
    std::vector<double> val(n, 1.0);
    for (int32_t i = 0; i <= n; ++i) rp[(size_t)i] = i;
    for (int32_t i = 0; i < n; ++i) ci[(size_t)i] = i;
    const std::vector<int64_t> nnz(nsys, n);
    const std::vector<const int32_t *> rps(nsys, rp.data()), cis(nsys, ci.data());
    const std::vector<const double *> vals(nsys, val.data());
    const std::vector<float> theta(kNParams, 0.0f);
    cg_fsai_trainer *t = nullptr;
    REQUIRE(cg_fsai_trainer_create(nsys, sizes.data(), nnz.data(), rps.data(), cis.data(), vals.data(), theta.data(),
                                   &t) == CG_OK, "%s", cg_last_error());
    std::vector<float> grad(kNParams);
    double loss = 0.0;
    auto step = [&](int32_t nsel, int32_t per) {
        return cg_fsai_loss_grad(t, nullptr, nsel, sys.data(), per, rows.data(), &loss, grad.data(), nullptr);
    };
    g_no_pinned = true;
    REQUIRE(step(4, 1024) == CG_ENOMEM, "no page-locked memory");   // the device buffer has grown
    g_no_pinned = false;
    REQUIRE(step(1, 16) == CG_OK && step(2, 512) == CG_OK && step(4, 1024) == CG_OK, "%s", cg_last_error());
    cg_fsai_trainer_destroy(t);
    REQUIRE(!g_overrun, "a step wrote past its page-locked buffer");
}

void check_abandoned() {
    const int32_t n = 8192;
    std::vector<int32_t> rp((size_t)n + 1), ci((size_t)n);
    std::vector<double> val((size_t)n, 2.0), b((size_t)n, 1.0), x((size_t)n, 0.0);
    for (int32_t i = 0; i <= n; ++i) rp[(size_t)i] = i;
    for (int32_t i = 0; i < n; ++i) ci[(size_t)i] = i;
    cg_handle *h = nullptr;
    REQUIRE(cg_create(n, n, rp.data(), ci.data(), val.data(), 0, n, &h) == CG_OK, "create");
    g_one_launch = true;
    cg_result res;
    const int rc = cg_solve(h, b.data(), x.data(), 1e-8, 10, &res);
    REQUIRE(rc == CG_OK && g_launches == 1, "%d: %s", rc, cg_last_error());
    cg_destroy(h);
}

void check_streams() {
    const int32_t n = 299521;
    const Matrix A = random_rows(n, n, 33);
    cg_handle *h = nullptr;
    REQUIRE(cg_create(n, (int64_t)A.ci.size(), A.rp.data(), A.ci.data(), A.val.data(), 0, n, &h) == CG_OK, "create");
    REQUIRE(h->A.use_st64, "no staged segments");
    ihipStream_t s[4], graph;
    graph.capture = true;
    std::vector<double> x((size_t)n, 1.0), y((size_t)n);
    auto on = [&](ihipStream_t &st) { REQUIRE(cg_set_stream(h, &st) == CG_OK, "set_stream"); };
    auto product = [&] { REQUIRE(cg_spmv(h, x.data(), y.data()) == CG_OK, "spmv"); };
    on(s[0]);
    product();
    product();
    REQUIRE(g_waits == 0, "%d waits on one stream", g_waits);
    on(s[3]);   // the solve without allocations: the wait alone
    cg_result res;
    REQUIRE(cg_solve_noalloc(h, x.data(), y.data(), 0.0, 1, &res) >= 0 && g_waits == 1 && g_events == 0,
            "%d waits, %d events: %s", g_waits, g_events, cg_last_error());
    on(s[0]);
    product();
    for (int k : {1, 0, 2, 2, 1}) {
        on(s[k]);
        product();
    }
    on(graph);   // an eager product is pending: a captured one leaves it so
    product();
    on(s[3]);
    REQUIRE(cg_solve(h, x.data(), y.data(), 0.0, 1, &res) >= 0, "solve");
    REQUIRE(g_fault.empty(), "%s", g_fault.c_str());
    cg_destroy(h);
}

}  // namespace

int main(int argc, char **argv) {
    const std::string what = argc > 1 ? argv[1] : "";
    if (what == "staged" && argc == 5) check_staged(std::atoi(argv[2]), std::atoi(argv[3]), std::atoi(argv[4]));
    else if (what == "widths") check_widths();
    else if (what == "mixed") check_mixed();
    else if (what == "stage") check_stage();
    else if (what == "abandoned") check_abandoned();
    else if (what == "streams") check_streams();
    else die("usage: host_checks staged ROWS COLS PER_ROW | widths | mixed | stage | abandoned | streams");
    std::printf("ok\n");
    return 0;
}
