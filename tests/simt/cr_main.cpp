// The plain conjugate residual solver on the host stand-in, with a diagonal H (test
// infrastructure).  Prints one line per check that fails; ends with "cr ok".
#include "../../paper_1611_06944_amd/csrc/solve_cr.hip"

#include <random>

namespace hdcr {

static std::vector<double> diag;  // H of the test, one value per complex entry
static int64_t applies = 0;
static int64_t odd_apply = 0;     // number of the apply that is scaled
static double odd_scale = 1.0;

int fail(int code, const std::string& msg) {
    fprintf(stderr, "%s\n", msg.c_str());
    return code;
}
template <typename T>
void launch_dslash(const FineGeom&, const C2<T>*, const C2<T>* in, C2<T>* out, hipStream_t) {
    const double f = ++applies == odd_apply ? odd_scale : 1.0;
    for (size_t i = 0; i < diag.size(); ++i) out[i] = make_double2(f * diag[i] * in[i].x, f * diag[i] * in[i].y);
}
template void launch_dslash<double>(const FineGeom&, const double2*, const double2*, double2*, hipStream_t);
int dslash_dots_blocks(const FineGeom&) { return 0; }
void launch_dslash_dots(const FineGeom&, const double2*, const double2*, double2*, const double2*, double*, hipStream_t) {
    abort();
}

struct Result {
    int code = 0;
    int64_t applies = 0;
    hdcr_solve_stats st = {};
    std::vector<double2> x;
    std::vector<double> hist;
};
static Result run(const std::vector<double2>& b, double tol, int maxiter, simt::Order order) {
    FineGeom g = {};
    g.N5 = (int)b.size() / 12;
    hdcr_solve_params prm = {};
    prm.tol = tol;
    prm.maxiter = maxiter;
    Result r;
    r.x.assign(b.size(), make_double2(0, 0));
    r.hist.assign(maxiter, 0.0);
    std::vector<char> work(cr_workspace_bytes(g) + 256);
    void* w = (void*)(((uintptr_t)work.data() + 255) & ~(uintptr_t)255);
    simt::order = order;
    applies = 0;
    r.code = cr_solve(g, &prm, nullptr, b.data(), r.x.data(), &r.st, r.hist.data(), maxiter, w, cr_workspace_bytes(g),
                      nullptr);
    r.applies = applies;
    r.hist.resize(r.st.history_len);
    return r;
}

static int failures = 0;
static void check(bool ok, const char* what, int tag = 0) {
    if (ok) return;
    ++failures;
    printf("failed: %s (%d)\n", what, tag);
}
static bool same(const Result& a, const Result& b) {
    return a.code == b.code && a.st.outer_iters == b.st.outer_iters && a.hist == b.hist &&
           memcmp(a.x.data(), b.x.data(), a.x.size() * sizeof(double2)) == 0;
}

}  // namespace hdcr

using namespace hdcr;

int main() {
    std::mt19937_64 rng(7);
    std::normal_distribution<double> gauss;
    std::uniform_real_distribution<double> uni(1.0, 2.0);
    // 128 workgroups, so that two wavefronts of each add up their partial sums
    const size_t n = 12 * 8192;
    std::vector<double2> b(n);
    diag.resize(n);
    for (size_t i = 0; i < n; ++i) {
        diag[i] = (i % 5 == 0 ? -1.0 : 1.0) * uni(rng);
        b[i] = make_double2(gauss(rng), gauss(rng));
    }
    // a workgroup that is late by a whole launch of the others takes the same decisions, at stops
    // after odd and even numbers of steps with a residual just below the tolerance
    const Result ref = run(b, 1e-30, 6, simt::IN_TURN);
    for (int k : {5, 6}) {
        const double tol = ref.hist[k - 1] * (1.0 + 1e-6);
        const Result a = run(b, tol, 100, simt::IN_TURN), c = run(b, tol, 100, simt::LATE);
        check(a.code == HDCR_OK && a.st.outer_iters == k, "the solve stops where it is to", k);
        check(same(a, c), "a late workgroup stops with the others", k);
        check(a.st.fine_applies_f64 == a.applies, "every application of H is counted", k);
    }
    // A second step (the third apply: H x, step 1, step 2) whose |Ap|^2 overflows or vanishes, though
    // its |Ar|^2 and <r, Ar> do not stop it: it changes nothing, x is the iterate of the first step.
    const Result one = run(b, 1e-30, 1, simt::IN_TURN);
    double arar = 0;  // |H r|^2 after the first step
    for (size_t i = 0; i < n; ++i) {
        const double rx = b[i].x - diag[i] * one.x[i].x, ry = b[i].y - diag[i] * one.x[i].y;
        arar += diag[i] * diag[i] * (rx * rx + ry * ry);
    }
    odd_apply = 3;
    odd_scale = sqrt(1.6e308 / arar);
    const Result big = run(b, 1e-30, 5, simt::IN_TURN);
    check(big.code == HDCR_ENAN && big.st.outer_iters == 1, "an overflow of |Ap|^2 ends the solve");
    check(memcmp(big.x.data(), one.x.data(), n * sizeof(double2)) == 0, "with the last good iterate");
    odd_scale = 1e-170;
    const Result small = run(b, 1e-30, 5, simt::IN_TURN);
    check(small.code == HDCR_EBREAKDOWN && small.st.outer_iters == 1, "a vanishing |Ap|^2 ends the solve");
    check(memcmp(small.x.data(), one.x.data(), n * sizeof(double2)) == 0, "with the last good iterate");
    odd_apply = 0;
    if (failures)
        printf("cr: %d failed\n", failures);
    else
        printf("cr ok\n");
    return failures != 0;
}
