// A run of steps with energies that fails at one of its launches: the rows of the steps
// before it are written all the same.  Argument: the bath (0: none, 2: Nose-Hoover).
// Every launch of a call of 40 steps fails once in turn.
#include "host_runtime.h"
#include "system.h"

using namespace rbsog;

int main(int argc, char **argv)
{
    if (argc != 2) return 2;
    const int bath = std::atoi(argv[1]);
    const int64_t N = 500;
    const int nsteps = 40;
    rbsog_sog sog{};
    rbsog_params p{};
    p.N = N;
    p.L = std::cbrt(4.0 * 3.141592653589793 * (double)N / 3.0);
    p.kT = 0.01;
    p.P = 50;
    p.seed = 3;
    p.precision = RBSOG_FP64;
    p.density = RBSOG_ADAPTIVE;
    p.skin = 0.1;
    size_t bytes = 0;
    if (rbsog_sog_init(2.0, 3.0, 1e-4, 1, RBSOG_AUTO, RBSOG_AUTO, &sog) != RBSOG_OK ||
        rbsog_workspace_size(&p, &sog, &bytes) != RBSOG_OK)
        return 2;
    void *ws = nullptr;
    double *x = nullptr, *one = nullptr, *rows = nullptr;
    if (hipMalloc(&ws, bytes) != hipSuccess || hipMalloc((void **)&x, 24 * N) != hipSuccess ||
        hipMalloc((void **)&one, 8 * N) != hipSuccess ||
        hipMalloc((void **)&rows, 8 * kEnergyCols * nsteps) != hipSuccess)
        return 2;
    for (int64_t i = 0; i < N; ++i) one[i] = 1.0;
    rbsog_handle *h = nullptr;
    if (rbsog_create(&p, &sog, one, one, ws, bytes, nullptr, &h) != RBSOG_OK) return 2;
    if (bath && rbsog_set_bath(h, bath, 1.0, 0.01) != RBSOG_OK) return 2;
    int evaluated = 0, moved = 0;   // steps up to their far field, and (global bath) up to their half-step
    std::vector<int> written(nsteps);
    host_runtime::on_launch = [&](const host_runtime::Launch &l) {
        if (l.name.find("k_far") != std::string::npos) ++evaluated;
        if (l.name.find("k_bath") != std::string::npos) moved += ((const BathArgs *)l.arg0)->mode & 2 ? 1 : 0;
        if (l.name.find("k_energy") != std::string::npos) {
            const EnergyArgs &a = *(const EnergyArgs *)l.arg0;
            const int64_t first = (a.out - rows) / kEnergyCols;
            for (int k = 0; k < a.rows; ++k) ++written.at((size_t)(first + k));
        }
    };
    int failures = 0, calls = 0;
    for (int at = 0;; ++at) {
        evaluated = moved = 0;
        written.assign(nsteps, 0);
        host_runtime::launches = 0;
        host_runtime::fail_launch = at;
        const int rc = rbsog_step(h, x, x, x, 0, nsteps, 0.01, rows);
        host_runtime::fail_launch = -1;
        const int done = bath ? moved : evaluated;
        for (int n = 0; n < nsteps; ++n)
            if (written[n] != (n < done ? 1 : 0)) {
                ++failures;
                std::printf("FAIL launch %d: %d steps done, row %d written %d times\n", at, done, n, written[n]);
                break;
            }
        ++calls;
        if (rc == RBSOG_OK) break;   // fewer launches than that
    }
    host_runtime::on_launch = nullptr;
    rbsog_destroy(h);
    std::printf("%d calls, %d failures\n", calls, failures);
    return failures != 0;
}
