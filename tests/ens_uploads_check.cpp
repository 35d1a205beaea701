// Admissions and the memory their uploads read from: what goes up has arrived when
// its source is changed or released, whether it fits the pinned memory or not, and
// nothing of the caller's is still being read when an admission returns, be it refused,
// failed or carried out.  Arguments: particle counts.
#include "host_runtime.h"
#include "system.h"

using namespace rbsog;

static int failures = 0;

static void expect(bool ok, int64_t N, const char *what)
{
    if (ok) return;
    ++failures;
    std::printf("FAIL N %lld: %s\n", (long long)N, what);
}

// the library's own memory, which it may go on reading from
static bool reads(const void *from, size_t bytes)
{
    for (const host_runtime::Copy &c : host_runtime::pending)
        if ((const char *)c.src < (const char *)from + bytes && (const char *)from < (const char *)c.src + c.bytes)
            return true;
    return false;
}

static void settle()
{
    host_runtime::carry_out(true, nullptr);
    host_runtime::stale = 0;
}

static void admissions(int64_t N)
{
    rbsog_sog sog{};
    rbsog_params p{};
    p.N = N;
    p.L = std::cbrt(4.0 * 3.141592653589793 * (double)N / 3.0);
    p.kT = 1.0;
    p.P = 50;
    p.seed = 3;
    p.precision = RBSOG_FP64;
    p.density = RBSOG_ADAPTIVE;
    p.skin = -1.0;
    size_t bytes = 0;
    if (rbsog_sog_init(2.0, 4.0, 1e-4, 1, RBSOG_AUTO, RBSOG_AUTO, &sog) != RBSOG_OK ||
        rbsog_ens_bytes(&p, &sog, 4, &bytes) != RBSOG_OK)
        std::exit(2);
    rbsog_ens *ens = nullptr;
    if (rbsog_ens_create(3 * bytes, 3, nullptr, &ens) != RBSOG_OK) std::exit(2);
    std::vector<double> x(3 * N, 1.0), v(3 * N, 0.5), q(N, 1.0), m(N, 1.0), zero(N, 0.0);
    const std::vector<double> *mine[] = {&x, &v, &q, &m, &zero};
    auto free_again = [&](const char *what) {
        for (const std::vector<double> *a : mine) expect(!reads(a->data(), 8 * a->size()), N, what);
    };
    int slot = -1;
    for (int k = 0; k < 2; ++k) {   // the second over the first's pinned memory
        x.assign(3 * N, 1.0 + k);
        expect(rbsog_ens_admit(ens, &p, &sog, x.data(), v.data(), q.data(), m.data(), 4, 0.01, &slot) == RBSOG_OK, N,
               "admission");
        free_again("an admission returns while its arrays are read");
    }
    host_runtime::carry_out(true, nullptr);
    expect(host_runtime::stale == 0, N, "a source changed before its copy was waited for");
    settle();
    // refused after its state has been sent
    expect(rbsog_ens_admit(ens, &p, &sog, x.data(), v.data(), zero.data(), m.data(), 4, 0.01, &slot) == RBSOG_EINVAL,
           N, "charges of zero are refused");
    free_again("a refused admission returns while its arrays are read");
    settle();
    // a launch that fails, at each of the admission's launches in turn
    for (int at = 0; at < 12; ++at) {
        host_runtime::launches = 0;
        host_runtime::fail_launch = at;
        const int rc = rbsog_ens_admit(ens, &p, &sog, x.data(), v.data(), q.data(), m.data(), 4, 0.01, &slot);
        host_runtime::fail_launch = -1;
        if (rc == RBSOG_OK) break;   // fewer launches than that
        expect(rc == RBSOG_EHIP, N, "a failed launch is reported");
        expect(host_runtime::waited_for_all(), N, "a failed admission returns its pool range with work in flight");
        free_again("a failed admission returns while its arrays are read");
        settle();
    }
    rbsog_ens_destroy(ens);
    settle();
}

int main(int argc, char **argv)
{
    // the copy kernel's pieces are read when something waits for them, like the runtime's copies
    host_runtime::on_launch = [](const host_runtime::Launch &l) {
        if (l.name.find("k_copy_segs") == std::string::npos) return;
        const CopySegs &a = *(const CopySegs *)l.arg0;
        for (int i = 0; i < a.n; ++i)
            if (a.s[i].kind == kCopyWords) {
                const char *src = (const char *)a.s[i].src;
                host_runtime::pending.push_back(
                    {a.s[i].dst, src, a.s[i].bytes, l.stream, std::vector<char>(src, src + a.s[i].bytes)});
            }
    };
    for (int i = 1; i < argc; ++i) admissions(std::atoll(argv[i]));
    std::printf("%d failures\n", failures);
    return failures != 0;
}
