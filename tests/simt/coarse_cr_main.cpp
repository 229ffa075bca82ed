// The coarse conjugate residual on the host stand-in (test infrastructure).  Prints one line per
// check that fails; ends with "coarse_cr ok".
#include "../../paper_1611_06944_amd/csrc/coarse.hip"

#include <random>

namespace hdcr {
// LDS of the kernels that take its size at launch
namespace {
alignas(16) thread_local unsigned char smem_raw[160 * 1024];
}

static CoarseGeom geom(int nb) {
    CoarseGeom c = {};
    const int C[4] = {2, 4, 4, 4};
    c.Nc = 1;
    for (int mu = 0; mu < 4; ++mu) {
        c.C[mu] = C[mu];
        c.cstride[mu] = c.Nc;
        c.Nc *= C[mu];
    }
    c.Nb = nb;
    c.nvec = nb / 2;
    return c;
}

// every buffer of a solve
struct Solve {
    std::vector<double2> r[2], Ar[2], Ap[2], p, x;
    std::vector<double> part, cs;
    std::vector<int> flags;
};
// all of maxiter steps enqueued, as the library does for a batch
static Solve run(const CoarseGeom& c, const std::vector<double2>& A, const std::vector<double2>& b, double tol,
                 int maxiter, simt::Order order) {
    const size_t n = b.size();
    Solve v;
    CoarseCRWork<double> w = {};
    for (int h = 0; h < 2; ++h) {
        v.r[h].assign(n, make_double2(0, 0));
        v.Ar[h] = v.Ap[h] = v.r[h];
        w.r[h] = v.r[h].data();
        w.Ar[h] = v.Ar[h].data();
        w.Ap[h] = v.Ap[h].data();
    }
    v.p = v.x = v.r[0];
    v.part.assign(CCR_START_PARTS + 10 * (size_t)ccr_groups<double>(c.Nc), 0.0);
    v.cs.assign(8, 0.0);
    v.flags.assign(CCR_FLAGS, 0);
    w.p = v.p.data();
    w.part = v.part.data();
    w.cs = v.cs.data();
    w.flags = v.flags.data();
    simt::order = order;
    launch_ccr_init<double>(c, b.data(), v.x.data(), w, maxiter, tol, nullptr);
    for (int k = 0; k <= maxiter; ++k) launch_ccr_step<double>(c, HDCR_C128, A.data(), v.x.data(), w, k, nullptr);
    return v;
}
static double norm(const std::vector<double2>& v) {
    double s = 0;
    for (const double2& e : v) s += e.x * e.x + e.y * e.y;
    return sqrt(s);
}
template <typename T> static bool same(const std::vector<T>& a, const std::vector<T>& b) {
    return memcmp(a.data(), b.data(), a.size() * sizeof(T)) == 0;
}

}  // namespace hdcr

using namespace hdcr;

int main() {
    int failures = 0;
    auto check = [&](bool ok, const char* what, int tag) {
        if (ok) return;
        ++failures;
        printf("failed: %s (%d)\n", what, tag);
    };
    const CoarseGeom c = geom(2);  // 128 workgroups: two wavefronts of each add up partial sums
    std::mt19937_64 rng(3);
    std::normal_distribution<double> gauss;
    const size_t n = (size_t)c.Nc * c.Nb;
    std::vector<double2> A(n * 9 * c.Nb, make_double2(0, 0)), b(n);
    for (int a = 0; a < c.Nc; ++a)  // diagonal blocks, well conditioned
        for (int k = 0; k < c.Nb; ++k) A[((size_t)a * 9 * c.Nb + k) * c.Nb + k].x = 1.5 + 0.5 * ((a * c.Nb + k) % 7) / 6.0;
    for (double2& e : b) e = make_double2(gauss(rng), gauss(rng));
    // A workgroup that is late by a whole launch of the others takes the same decisions, at stops
    // after odd and even numbers of steps with a residual just below the tolerance.
    for (int k : {3, 4}) {
        const Solve ref = run(c, A, b, 0.0, k, simt::IN_TURN);
        const double tol = norm(ref.r[k & 1]) / norm(b) * (1.0 + 1e-6);
        const Solve s = run(c, A, b, tol, k + 2, simt::IN_TURN), t = run(c, A, b, tol, k + 2, simt::LATE);
        check(same(s.x, ref.x), "the solve stops where it is to", k);
        check(same(t.x, s.x) && same(t.p, s.p) && same(t.flags, s.flags), "a late workgroup stops with the others", k);
        for (int h = 0; h < 2; ++h)
            check(same(t.r[h], s.r[h]) && same(t.Ar[h], s.Ar[h]) && same(t.Ap[h], s.Ap[h]), "and changes nothing", k);
    }
    if (failures)
        printf("coarse_cr: %d failed\n", failures);
    else
        printf("coarse_cr ok\n");
    return failures != 0;
}
