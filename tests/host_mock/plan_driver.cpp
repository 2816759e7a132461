// Host code of matrix creation and of the solvers against the mock HIP
// runtime; the first argument names the check.  Prints what was found and
// exits 0 when the check holds.
#include <dlfcn.h>
#include <pthread.h>
#include <sys/resource.h>

#include <algorithm>
#include <atomic>
#include <climits>
#include <cstdint>
#include <cstdlib>
#include <new>
#include <cstdio>
#include <cstring>
#include <string>
#include <thread>
#include <utility>
#include <vector>

#include "internal.h"
#include "spmv.h"

extern "C" const char *mock_launch_log(void);

// Device memory as the runtime reports it.
static size_t mem_free = 0, mem_total = 0;
extern "C" int hipMemGetInfo(size_t *free, size_t *total) {
    *free = mem_free ? mem_free : size_t(1) << 40;
    *total = mem_total ? mem_total : size_t(1) << 40;
    return 0;
}

// The countdown-th allocation of this thread from now on fails (0: none).
static thread_local long fail_at = 0;
static void *allocate(size_t n) {
    if (fail_at > 0 && --fail_at == 0) return nullptr;
    return std::malloc(n ? n : 1);
}
void *operator new(size_t n) {
    void *p = allocate(n);
    if (!p) throw std::bad_alloc();
    return p;
}
void *operator new(size_t n, const std::nothrow_t &) noexcept { return allocate(n); }
void operator delete(void *p) noexcept { std::free(p); }
void operator delete(void *p, size_t) noexcept { std::free(p); }

// Threads started while the library's capture gate was held.
static std::atomic<int> started{0}, under_gate{0};

struct Start {
    void *(*f)(void *);
    void *arg;
    std::atomic<bool> looked{false};
};

static void *look_at_gate(void *p) {
    Start *s = static_cast<Start *>(p);
    void *(*f)(void *) = s->f, *arg = s->arg;
    if (spmvlib::capture_gate().try_lock()) spmvlib::capture_gate().unlock();
    else ++under_gate;
    s->looked = true;
    return f(arg);
}

// Every thread of the process starts here; the caller waits until it has looked.
extern "C" int pthread_create(pthread_t *t, const pthread_attr_t *a, void *(*f)(void *), void *arg) {
    static const auto real = reinterpret_cast<int (*)(pthread_t *, const pthread_attr_t *, void *(*)(void *), void *)>(
        dlsym(RTLD_NEXT, "pthread_create"));
    Start s{f, arg};
    const int rc = real(t, a, look_at_gate, &s);
    ++started;
    while (rc == 0 && !s.looked) std::this_thread::yield();
    return rc;
}

namespace {

struct Csr {
    int32_t n = 0, n_cols = 0;
    std::vector<int32_t> row_ptr{0}, col;
    std::vector<double> val;
    void row(std::initializer_list<int32_t> c) {
        for (int32_t v : c) col.push_back(v);
        end_row();
    }
    void end_row() {
        ++n;
        row_ptr.push_back((int32_t)col.size());
        val.resize(col.size(), 1.0);
    }
    int create(const spmv_params *p, uint32_t flags, spmv_matrix **out) const {
        return spmv_create(n, n_cols, (int64_t)col.size(), row_ptr.data(), col.data(), val.data(), flags, p, out);
    }
};

int failures = 0;
void check(bool ok, const char *what) {
    std::printf("%s %s\n", ok ? "ok" : "FAIL", what);
    if (!ok) {
        std::printf("  last error: %s\n", spmv_last_error());
        ++failures;
    }
}

// The served solver modes capture their iterations (the mock answers the
// host's read of the scalar state, 96 bytes, with a converged solve).
void solves_capture() {
    Csr A;
    A.n_cols = 300;
    for (int32_t i = 0; i < 300; ++i) {
        if (i > 0) A.col.push_back(i - 1);
        A.col.push_back(i);
        A.end_row();
    }
    spmv_matrix *M = nullptr;
    check(A.create(nullptr, SPMV_VALUES_FP32 | SPMV_VALUES_BF16, &M) == SPMV_OK, "create");
    std::vector<double> b(300, 1.0), x(300, 0.0);
    for (int mode : {CG_FP64, CG_MIXED_FP32}) {
        (void)mock_launch_log();
        cg_info info{};
        // the mixed solve's outer residual stays where the mock put it
        const int rc = cg_solve(M, b.data(), x.data(), 1e-8, 100, mode, &info, nullptr);
        check(rc == (mode == CG_FP64 ? SPMV_OK : SPMV_ENOTCONV), "cg_solve");
        check(std::string(mock_launch_log()).find("k_update_xpr") != std::string::npos, "iterations launched");
        check(info.iterations > 0, "iterations counted");
    }
    spmv_destroy(M);
}

// Sweep tiles beside long rows: whole rounds of workgroups while the tiles
// stay large, row tiles where they do not.
void sweep_rounds() {
    constexpr int kCus = 256, kLong = 1021, kRows = 1'000'000, kPerRow = 7;
    uint32_t lcg = 1;
    std::vector<int32_t> row_ptr, col;
    for (const auto &[n_long, taken] : {std::pair{0, true}, {1, true}, {8, true}, {64, true}, {512, false}, {8192, false}}) {
        row_ptr.assign(1, 0);
        col.clear();
        for (int r = 0, next = 0; r < kRows; ++r) {
            int len = kPerRow;
            if (next < n_long && r == (int)((int64_t)(next + 1) * kRows / (n_long + 1))) {
                len = kLong + 1;
                ++next;
            }
            for (int k = 0; k < len; ++k) {
                lcg = lcg * 1664525u + 1013904223u;
                col.push_back((int32_t)((uint64_t)lcg * kRows >> 32));
            }
            row_ptr.push_back((int32_t)col.size());
        }
        spmvlib::SweepPlan S;
        const bool built = spmvlib::build_sweep_plan(kRows, kRows, row_ptr.data(), col.data(), kLong, kCus, S);
        const std::string what = std::to_string(n_long) + " long rows";
        check(built == taken, (what + ": taken or left as expected").c_str());
        if (!built) continue;
        const int tiles = (int)(S.bound.size() / 2);
        std::printf("  %d tiles, width %d\n", tiles, S.width);
        check(tiles <= 2 * kCus, (what + ": two rounds of workgroups").c_str());
        check(S.width <= spmvlib::kSweepTile, (what + ": tiles fit the LDS").c_str());
        // every row that is not long in one tile, in order
        int64_t rows = 0;
        for (int t = 0; t < tiles; ++t) rows += S.bound[2 * t + 1] - S.bound[2 * t];
        check(rows == kRows - n_long, (what + ": every other row in a tile").c_str());
    }
    // a run that ends in empty rows, and runs of empty rows alone
    std::vector<int> lens(800'000, 6);
    std::fill(lens.end() - 1000, lens.end(), 0);
    for (int r : {1000, 1002, 1004}) lens[r] = 2000;
    lens[1001] = lens[1003] = 0;
    row_ptr.assign(1, 0);
    col.clear();
    for (int len : lens) {
        for (int k = 0; k < len; ++k) {
            lcg = lcg * 1664525u + 1013904223u;
            col.push_back((int32_t)((uint64_t)lcg * kRows >> 32));
        }
        row_ptr.push_back((int32_t)col.size());
    }
    spmvlib::SweepPlan S;
    check(spmvlib::build_sweep_plan((int)lens.size(), kRows, row_ptr.data(), col.data(), kLong, kCus, S), "empty rows");
    check(S.bound.size() / 2 <= kCus, "empty rows: one round of workgroups");
}

// 4,200 tiles' worth of a banded matrix, its columns `shift` to the right.
Csr banded(int32_t n, int32_t n_cols, int32_t shift) {
    Csr A;
    A.n_cols = n_cols;
    for (int32_t i = 0; i < n; ++i) {
        for (int32_t d = 0; d < 18; ++d) A.col.push_back(shift + std::min(i + d, n - 1));
        A.end_row();
    }
    return A;
}

// The plan's memory follows the matrix's entries, not its number of columns.
void wide_matrix() {
    const int32_t n = 70'000, n_cols = INT32_MAX;
    const Csr A = banded(n, n_cols, n_cols - n);
    spmv_matrix *M = nullptr;
    spmv_info info{};
    check(A.create(nullptr, 0, &M) == SPMV_OK && spmv_get_info(M, &info) == SPMV_OK, "create");
    check(info.device_bytes > 20 * info.nnz, "the layout of its products is there");
    rusage u{};
    getrusage(RUSAGE_SELF, &u);
    std::printf("  peak %ld MB\n", u.ru_maxrss / 1024);
    check(u.ru_maxrss < 1024 * 1024, "peak host memory below 1 GB");
    spmv_destroy(M);
}

// A layout's host work keeps no solve of another thread from its capture.
void plans_without_gate() {
    const Csr A = banded(120'000, 120'000, 0);
    spmv_matrix *M = nullptr;
    spmv_info info{};
    check(A.create(nullptr, 0, &M) == SPMV_OK && spmv_get_info(M, &info) == SPMV_OK, "create");
    check(info.device_bytes > 20 * info.nnz, "the layout of its products is there");
    std::printf("  %d threads started, %d while the gate was held\n", started.load(), under_gate.load());
    check(started > 0 && under_gate == 0, "no thread started while the gate was held");
    spmv_destroy(M);
}

// A layout is added only while half of the device's memory stays free.
void layout_memory() {
    const Csr A = banded(70'000, 70'000, 0);
    mem_total = size_t(1) << 30;
    int64_t bytes[4];
    const size_t frees[4] = {size_t(1) << 30, (size_t(1) << 29) + (size_t(9) << 20), (size_t(1) << 29) + (size_t(16) << 20), 1};
    for (int i = 0; i < 4; ++i) {
        mem_free = frees[i];
        spmv_matrix *M = nullptr;
        spmv_info info{};
        check(A.create(nullptr, 0, &M) == SPMV_OK && spmv_get_info(M, &info) == SPMV_OK, "create");
        bytes[i] = info.device_bytes;
        std::printf("  free %zu MB: %lld bytes\n", frees[i] >> 20, (long long)bytes[i]);
        spmv_destroy(M);
    }
    // 12.1 MB of layout
    check(bytes[0] > 20 * (int64_t)A.col.size() && bytes[2] == bytes[0], "a layout where there is room");
    check(bytes[1] < 13 * (int64_t)A.col.size() && bytes[3] == bytes[1], "none where half would not stay free");
}

// A served matrix takes no more than the server counted for it: a budget of
// exactly that and one request's vectors serves it again and again.
void served_budget() {
    Csr A;  // one entry a row: the most tiles per entry
    A.n_cols = 200'000;
    for (int32_t i = 0; i < A.n_cols; ++i) A.row({i});
    const uint64_t n = (uint64_t)A.n, padded = n + 16;  // entries and the arrays' padding
    srv_config cfg{};
    cfg.n_slots = 1;
    cfg.hbm_budget_bytes = 4 * (n + 1) + 12 * padded + 64 * (n / 512 + 16) + 16 * n;
    spmv_server *S = nullptr;
    int32_t id = -1;
    check(srv_create(&cfg, &S) == SPMV_OK, "server");
    check(srv_add_matrix(S, A.n, A.n_cols, (int64_t)n, A.row_ptr.data(), A.col.data(), A.val.data(), &id) == SPMV_OK, "matrix");
    std::vector<double> x(n, 1.0), y(n);
    for (int i = 0; i < 3; ++i) {
        uint64_t ticket = 0;
        srv_result r{};
        check(srv_submit(S, id, SRV_SPMV, 1, x.data(), y.data(), 0.0, 0, &ticket) == SPMV_OK, "submit");
        (void)srv_wait(S, ticket, &r);
        check(r.done && r.status == SPMV_OK, (std::string("request served ") + r.message).c_str());
    }
    srv_stats st{};
    (void)srv_get_stats(S, &st);
    std::printf("  used %lld of %llu bytes\n", (long long)st.used_bytes, (unsigned long long)cfg.hbm_budget_bytes);
    (void)srv_destroy(S);
}

// An allocation that fails anywhere in a creation (on the calling thread) is
// SPMV_ENOMEM, or a handle without its second layout; no exception comes out.
void creation_without_memory() {
    const Csr jag = banded(62'000, 62'000, 0);
    Csr rest = banded(4'000, 4'000, 0);  // rows cut to the k-vector product's tiles, and a long row
    for (int k = 0; k < 5000; ++k) rest.col.push_back(k % 4000);
    rest.end_row();
    spmv_params wide{};
    wide.tile_nnz = 4096;
    for (const Csr *A : {&jag, (const Csr *)&rest}) {
        const spmv_params *p = A == &jag ? nullptr : &wide;
        int failed = 0, thrown = 0, other = 0, n = 1;
        for (bool done = false; !done; ++n) {
            spmv_matrix *M = nullptr;
            int rc = SPMV_OK;
            fail_at = n;
            try {
                rc = A->create(p, SPMV_VALUES_FP32, &M);
            } catch (const std::exception &) {
                ++thrown;
                rc = SPMV_ENOMEM;
            }
            done = fail_at > 0;  // more than the creation makes
            fail_at = 0;
            if (rc == SPMV_ENOMEM) ++failed;
            else if (rc != SPMV_OK) ++other;
            if (rc != SPMV_OK && M) ++other;
            if (M) spmv_destroy(M);
        }
        std::printf("  %d allocations, %d failed creations, %d exceptions\n", n - 2, failed, thrown);
        check(failed > 0 && thrown == 0 && other == 0, "no exception leaves spmv_create");
    }
}

}  // namespace

int main(int argc, char **argv) {
    const std::string what = argc > 1 ? argv[1] : "";
    if (what == "solves_capture") solves_capture();
    else if (what == "sweep_rounds") sweep_rounds();
    else if (what == "wide_matrix") wide_matrix();
    else if (what == "plans_without_gate") plans_without_gate();
    else if (what == "layout_memory") layout_memory();
    else if (what == "served_budget") served_budget();
    else if (what == "creation_without_memory") creation_without_memory();
    else ++failures;
    return failures ? 1 : 0;
}
