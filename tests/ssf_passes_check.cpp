// rbsog_ssf over its passes: every call that its contract takes is carried out, and
// every launch of partial sums stays within the staging area and the partials'
// buffer of the scratch.  Arguments: N m_s pairs.
#include "host_runtime.h"
#include "system.h"

using namespace rbsog;

int main(int argc, char **argv)
{
    int failures = 0;
    for (int i = 1; i + 1 < argc; i += 2) {
        const int64_t N = std::atoll(argv[i]);
        const int m_s = std::atoi(argv[i + 1]);
        size_t bytes = 0;
        if (rbsog_ssf_scratch_size(N, m_s, &bytes) != RBSOG_OK) return 2;
        char *scratch = nullptr;
        if (hipMalloc((void **)&scratch, bytes) != hipSuccess) return 2;
        int64_t modes = 0;
        int bad = 0;
        host_runtime::on_launch = [&](const host_runtime::Launch &l) {
            if (l.name.find("k_rho_partial") == std::string::npos) return;
            const RhoArgs &a = *(const RhoArgs *)l.arg0;
            modes += a.P;
            const char *end = (const char *)(a.part + (size_t)a.nchunk * a.P);
            if ((255 / a.P + 2) * a.chunk > kRhoStage || (int64_t)a.nchunk * a.chunk < N || end > scratch + bytes ||
                (int64_t)l.grid.x * kBlock < (int64_t)a.nchunk * a.P)
                ++bad;
        };
        static double x[1], s[1];
        const int rc = rbsog_ssf(N, 10.0, x, x, m_s, scratch, bytes, nullptr, s);
        if (rc != RBSOG_OK || bad || modes != lattice_points(m_s)) {
            ++failures;
            std::printf("FAIL N %lld m_s %d: status %d (%s), %lld of %lld modes, %d launches out of bounds\n",
                        (long long)N, m_s, rc, rc ? rbsog_last_error() : "", (long long)modes,
                        (long long)lattice_points(m_s), bad);
        }
        host_runtime::on_launch = nullptr;
        hipFree(scratch);
    }
    std::printf("%d failures\n", failures);
    return failures != 0;
}
