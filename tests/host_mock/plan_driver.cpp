// Host code of matrix creation and of the solvers against the mock HIP
// runtime; the first argument names the check.  Prints what was found and
// exits 0 when the check holds.
#include <cstdio>
#include <cstring>
#include <string>
#include <vector>

#include "spmv.h"

extern "C" const char *mock_launch_log(void);

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

}  // namespace

int main(int argc, char **argv) {
    const std::string what = argc > 1 ? argv[1] : "";
    if (what == "solves_capture") solves_capture();
    else ++failures;
    return failures ? 1 : 0;
}
