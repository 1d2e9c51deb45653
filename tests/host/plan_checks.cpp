// Checks of the plan's host arithmetic (tables, LDS layouts, dispatch rules)
// against what the kernels do with it.  No device is touched.  Each check
// prints what fails and returns the number of failures.
#ifndef BSDE_CAPI
#define BSDE_CAPI "../../paper_1909_13560_amd/csrc/capi.hip"
#endif
#include BSDE_CAPI

namespace {

int fails = 0;
#define EXPECT(c, ...)                          \
    do {                                        \
        if (!(c)) {                             \
            if (++fails <= 10) {                \
                std::printf("failed: %s: ", #c); \
                std::printf(__VA_ARGS__);       \
                std::printf("\n");              \
            }                                   \
        }                                       \
    } while (0)

constexpr size_t kLds = 163840;  // LDS per block

// K = k steps of dt = 1 / 64 on nx points, dx = 1, so that vol sqrt(2 dt) = R
// and drift dt = cells
bsde_problem problem(int nx, int k, int L, double R, double cells, int n_t = 64)
{
    bsde_problem p;
    std::memset(&p, 0, sizeof(p));
    p.d = 1;
    p.T = n_t / 64.0;
    p.n_t = n_t;
    p.k_y = p.k_z = k;
    p.L = L;
    p.n_x[0] = nx;
    p.x_min[0] = 0.0;
    p.x_max[0] = nx - 1.0;
    p.vol[0][0] = R * std::sqrt(32.0);
    p.drift[0] = 64.0 * cells;
    p.driver = BSDE_DRIVER_LINEAR;
    p.p[0] = -0.05;
    p.p[1] = -0.2;
    p.picard_max = 30;
    return p;
}

// Exact expectations on B-spline coefficients: a point that takes the end
// corrections of layer n+1 finds both end coefficients in its block's window
// (the kernel keeps only what the window holds), and every point whose basis
// functions reach over an end takes them.
int check_exact_ends()
{
    const int T = bsde::kExactTile;
    for (int nx : {4, 5, 63, 64, 65, 66, 127, 128, 129, 193, 700})
        for (int k : {1, 3, 6})
            for (double R : {0.5, 3.0, 9.0})
                for (double cells = -130.0; cells <= 130.0; cells += 6.5)
                    for (int G : {1, 2}) {
                        bsde_problem p = problem(nx, k, 8, R, cells);
                        p.quad = BSDE_QUAD_EXACT;
                        Instance in;
                        EXPECT(build_instance(p, in), "n_x %d", nx);
                        const ExactLds l = exact_layout(in, G);
                        for (int i = 0; i < nx; ++i) {
                            const int lo = i / T * T + l.lo[1], hi = lo + l.W[1];  // records [lo, hi)
                            if (i < in.ex_nl[1])
                                EXPECT(lo <= 0 && 1 < hi, "n_x %d K %d R %g drift %g point %d: left end", nx,
                                       k, R, cells, i);
                            if (nx - 1 - i < in.ex_nr[1])
                                EXPECT(lo <= nx - 2 && nx - 1 < hi,
                                       "n_x %d K %d R %g drift %g point %d: right end", nx, k, R, cells, i);
                        }
                        for (int j = 1; j <= k; ++j) {
                            const bsde::GaussBand &b = in.band[j];
                            const int cells_j = (int)b.i0.size();
                            auto reached = [&](int c) { return c >= b.klo && c < b.klo + cells_j; };
                            for (int i = 0; i < nx; ++i) {
                                const int q = nx - 1 - i;
                                const bool left = reached(-1 - i) || reached(-i);
                                const bool right = reached(q) || reached(q - 1);
                                EXPECT(!left || i < in.ex_nl[j], "n_x %d layer %d point %d", nx, j, i);
                                EXPECT(!right || q < in.ex_nr[j], "n_x %d layer %d point %d", nx, j, i);
                            }
                        }
                    }
    return fails;
}

}  // namespace

int main(int argc, char **argv)
{
    const std::string what = argc > 1 ? argv[1] : "";
    if (what == "exact_ends") return check_exact_ends() != 0;
    std::printf("unknown check\n");
    return 2;
}
