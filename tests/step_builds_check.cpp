// Which build the steps of a system of N particles take: one launch of one workgroup,
// or three passes.  Rebuilds are played by raising the device's count: `every` steps
// once (0: never).  Arguments: N every skin(< 0: the default).  Prints, per call of 20
// steps, the steps built by one workgroup and those by the passes.
#include "host_runtime.h"
#include "system.h"

using namespace rbsog;

int main(int argc, char **argv)
{
    if (argc != 4) return 2;
    const int64_t N = std::atoll(argv[1]);
    const int every = std::atoi(argv[2]);
    rbsog_sog sog{};
    rbsog_params p{};
    p.N = N;
    p.L = std::cbrt(4.0 * 3.141592653589793 * (double)N / 3.0);
    p.kT = 0.01;
    p.P = 50;
    p.seed = 3;
    p.precision = RBSOG_FP64;
    p.density = RBSOG_ADAPTIVE;
    p.skin = std::atof(argv[3]);
    size_t bytes = 0;
    if (rbsog_sog_init(2.0, 4.0, 1e-4, 1, RBSOG_AUTO, RBSOG_AUTO, &sog) != RBSOG_OK ||
        rbsog_workspace_size(&p, &sog, &bytes) != RBSOG_OK)
        return 2;
    void *ws = nullptr;
    double *x = nullptr, *one = nullptr;
    if (hipMalloc(&ws, bytes) != hipSuccess || hipMalloc((void **)&x, 24 * N) != hipSuccess ||
        hipMalloc((void **)&one, 8 * N) != hipSuccess)
        return 2;
    for (int64_t i = 0; i < N; ++i) one[i] = 1.0;
    rbsog_handle *h = nullptr;
    if (rbsog_create(&p, &sog, one, one, ws, bytes, nullptr, &h) != RBSOG_OK) return 2;
    int small = 0, passes = 0, steps = 0;
    host_runtime::on_launch = [&](const host_runtime::Launch &l) {
        if (l.name.find("k_build_small") != std::string::npos) ++small;
        if (l.name.find("k_cell_ids") != std::string::npos) ++passes;
        if (l.name.find("k_far") != std::string::npos) {
            const FarArgs &a = *(const FarArgs *)l.arg0;
            if (every > 0 && ++steps % every == 0 && a.rebuilds) *a.rebuilds += 1;
        }
    };
    for (int call = 0; call < 4; ++call) {
        small = passes = 0;
        if (rbsog_step(h, x, x, x, 20 * call, 20, 0.01, nullptr) != RBSOG_OK) return 2;
        std::printf("%d %d\n", small, passes);
    }
    host_runtime::on_launch = nullptr;
    rbsog_destroy(h);
    return 0;
}
