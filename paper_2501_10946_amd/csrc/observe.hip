// Observables of Section 5.1 on the device: the static structure factor by
// lattice shell (computed with the structure-factor kernels of the far field
// over every mode of the shells), the pair-distance histogram behind the
// radial distribution function (over the fine cell grid of a system), and the
// unwrapped displacements behind the mean squared displacement with the
// velocity autocorrelation.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <vector>

#include "dev_common.h"
#include "dev_window.h"
#include "system.h"

namespace rbsog {
namespace {

// The partial sums of a pass share a buffer sized for passes of kSsfModes modes
// with the groups a launch of their own takes; larger groups make room for more
// modes, and fewer passes (each two launches) follow.
constexpr int kSsfModes = 1024;

struct SsfPlan {
    int64_t K;       // modes with 1 <= |n|^2 <= m_s
    int P;           // modes per pass that the partial buffer is sized for
    int pass, chunk; // modes per pass, particles per group
    size_t o_tab, o_modes, o_rho, o_start, o_part, total;
};

// partial sums of a pass of P modes: its particle groups times P
size_t ssf_partials(int64_t N, int P)
{
    const int c = rho_chunk((int)N, P);
    return (size_t)((N + c - 1) / c) * (size_t)P;
}

SsfPlan ssf_plan(int64_t N, int m_s)
{
    SsfPlan p{};
    p.K = lattice_points(m_s);
    p.P = (int)std::max<int64_t>(1, std::min<int64_t>(p.K, kSsfModes));
    const int rest = (int)(p.K % p.P);
    const size_t npart = std::max(ssf_partials(N, p.P), rest ? ssf_partials(N, rest) : (size_t)0);
    size_t off = 0;
    auto take = [&](size_t bytes) {
        size_t o = off;
        off = align_up(off + bytes);
        return o;
    };
    p.o_tab = take(sizeof(double2) * kPhaseTable);
    p.o_modes = take(sizeof(double4) * (size_t)std::max<int64_t>(p.K, 1));
    p.o_rho = take(sizeof(double2) * (size_t)std::max<int64_t>(p.K, 1));
    // not used: the size that callers have asked for stays what it was
    take(sizeof(double2) * (size_t)p.P);
    take(sizeof(double) * (size_t)p.P);
    p.o_start = take(sizeof(int64_t) * ((size_t)m_s + 2));
    p.o_part = take(sizeof(double2) * npart);
    p.total = off;
    // the group size that needs the fewest passes (the smallest of those: more
    // workgroups), its passes of one size
    p.pass = p.P;
    p.chunk = rho_chunk((int)N, p.P);
    int64_t passes = (p.K + p.P - 1) / p.P;
    for (int c = p.chunk; 2 * c <= kRhoChunkMax && passes > 1;) {
        c *= 2;
        const int64_t fit = (int64_t)(npart / (size_t)((N + c - 1) / c));
        const int64_t n = fit < p.P ? passes : (p.K + fit - 1) / fit;
        if (n >= passes) continue;
        passes = n;
        p.pass = (int)((p.K + n - 1) / n);
        p.chunk = c;
    }
    return p;
}

// s[m] = mean over the modes of shell m of |rho|^2: one wave per shell, lane l the
// modes l, l + 64, ... in order, the lanes added by a fixed butterfly (a thread
// per shell waited for one load after the other: 4 168 modes in 100 shells 23 us)
__global__ __launch_bounds__(kBlock) void k_ssf_shells(const double2 *__restrict__ rho,
                                                       const int64_t *__restrict__ start, int m_s,
                                                       double *__restrict__ s)
{
    const int m = blockIdx.x * (kBlock / 64) + (threadIdx.x >> 6), lane = threadIdx.x & 63;
    if (m > m_s) return;   // whole waves
    const int64_t a = start[m], b = start[m + 1];
    double acc = 0.0;
    for (int64_t p = a + lane; p < b; p += 64) acc += rho[p].x * rho[p].x + rho[p].y * rho[p].y;
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) acc += __shfl_xor(acc, off);
    if (lane == 0) s[m] = b > a ? acc / (double)(b - a) : 0.0;
}

// ---------------------------------------------------------------------------
// pair-distance histogram
// ---------------------------------------------------------------------------

struct RdfArgs {
    int nbins;
    CellGeom g;               // the fine grid: cells >= r_max / 2 wide, 5 x 5 x 5 stencil
    double w[3];              // its cell widths
    const double4 *xs;        // cell order
    const int32_t *cell_start;
    int own;                  // passes of a cell pair that its own wave takes
    double rmax2, dr;
    unsigned long long *hist;
};

constexpr int kRdfMaxBins = 4096;
constexpr int kRdfThreads = 512;
constexpr int kRdfWaves = kRdfThreads / 64;
constexpr int kRdfHomes = 16;      // home particles per pass over a window
constexpr int kRdfBlocks = 768;    // three per compute unit: what LDS holds up to ~1000 bins

// Adds the counted distances queue[0 .. n), n <= 64, to the workgroup's bins.
__device__ inline void rdf_count(const RdfArgs &a, const double *queue, int n, unsigned long long *h)
{
    const int lane = threadIdx.x & 63;
    if (lane < n) {
        int b = (int)floor(sqrt(queue[lane]) / a.dr);
        if (b >= a.nbins) b = a.nbins - 1;
        atomicAdd(&h[b], 1ull);
    }
}

// A wave's 64 candidates from c0 on, image-shifted (the origin past the last).
struct RdfChunk {
    double x, y, z;
};
__device__ inline RdfChunk rdf_chunk(const RdfArgs &a, const PairTables &w, const uint8_t *pidx, bool tabled, int c0,
                                     int total)
{
    const int c = c0 + (int)(threadIdx.x & 63);
    RdfChunk o{0.0, 0.0, 0.0};
    if (c < total) {
        const int l = tabled ? (int)pidx[c] : window_piece(w.pref, c);
        const double4 r = a.xs[w.first[l] + c];
        o.x = r.x + w.shift[0][l];
        o.y = r.y + w.shift[1][l];
        o.z = r.z + w.shift[2][l];
    }
    return o;
}

// One wave's work on cell pair q, as the list build does it: the candidates of the pair's
// 5 x 5 x 6-cell window 64 at a time (image-shifted, each neighbour within r_max <= L/3
// met once) against the pair's home particles, kRdfHomes per pass over the window: the
// passes first, first + step, ... before end.  The squared distances below r_max^2 (a
// fifth or so) are queued in LDS and binned 64 at a time, so that the square root and the
// division run on full waves.
__device__ inline void rdf_pair(const RdfArgs &a, int q, int first, int step, int end, PairTables &w, double4 *home,
                                double *qu, uint8_t *pidx, unsigned long long *h, int &queued)
{
    const int lane = threadIdx.x & 63;
    PairWindow win;
    double centre[3];
    if (!pair_window<false>(a.g, a.w, a.cell_start, q, w, centre, win)) return;   // uniform
    const int total = win.total;
    const bool tabled = window_pieces(w, total, pidx);
    const int home_c = win.h_beg - __builtin_amdgcn_readfirstlane(w.first[pair_window_home_piece(a.g, q)]);
    const int passes = min(end, (win.h_end - win.h_beg + kRdfHomes - 1) / kRdfHomes);
    for (int p = first; p < passes; p += step) {
        const int hb = win.h_beg + p * kRdfHomes;
        const int nh = min(kRdfHomes, win.h_end - hb);   // uniform
        if (lane < nh) home[lane] = a.xs[hb + lane];
        wave_lds_fence();
        const int hc = home_c + (hb - win.h_beg);   // candidate index of the pass's first home
        // the next 64 candidates load while these are tested
        RdfChunk next = rdf_chunk(a, w, pidx, tabled, 0, total);
        for (int c0 = 0; c0 < total; c0 += 64) {
            const RdfChunk cur = next;
            if (c0 + 64 < total) next = rdf_chunk(a, w, pidx, tabled, c0 + 64, total);
            const uint64_t live = __builtin_amdgcn_ballot_w64(c0 + lane < total);
            const int own = c0 + lane - hc;   // the pass's home this lane holds (any other value: none)
            for (int hp = 0; hp < nh; hp += 2) {   // two at a time: their LDS reads overlap
                const double4 r[2] = {home[hp], home[min(hp + 1, nh - 1)]};
#pragma unroll
                for (int i = 0; i < 2; ++i) {
                    if (hp + i >= nh) break;   // uniform
                    const double ux = r[i].x - cur.x, uy = r[i].y - cur.y, uz = r[i].z - cur.z;
                    const double r2 = fma(uz, uz, fma(ux, ux, uy * uy));
                    const uint64_t m = __builtin_amdgcn_ballot_w64(r2 < a.rmax2) & live &
                                       __builtin_amdgcn_ballot_w64(own != hp + i);
                    const uint32_t k = __builtin_amdgcn_mbcnt_hi(
                        (uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, (uint32_t)queued));
                    if (__builtin_amdgcn_inverse_ballot_w64(m)) qu[k] = r2;   // queued < 64: k < 128
                    queued += __popcll(m);
                    if (queued >= 64) {   // uniform
                        wave_lds_fence();
                        rdf_count(a, qu, 64, h);
                        queued -= 64;
                        const double rest = qu[64 + lane];
                        wave_lds_fence();
                        qu[lane] = rest;   // those past `queued` are written over
                        wave_lds_fence();
                    }
                }
            }
        }
        wave_lds_fence();   // the next pass overwrites the homes
    }
}

// The cell pairs of the fine grid are dealt to the waves in turn, each with its first
// passes (a.own: what nearly every pair of a uniform system needs).  The passes that are
// left in crowded pairs are dealt to kRdfSlices waves: each looks through a share of the
// pairs, spread over the grid, a lane per pair, and takes its turn.  A workgroup's counts go through LDS,
// then one atomic add per non-empty bin.  Integer counts: the result does not depend on
// the order of the additions.
//
// One particle per thread walking its own 125 cells left most lanes idle at the
// ends of cells of ~3 particles and divided on the lanes that passed: N = 2e5, r_max
// = 4, 200 bins took 307 us, this takes 121 (vector instructions issue in half of
// its cycles; the latency of the window tables takes most of the rest).  Dealt by whole
// pairs, neighbouring pairs to a workgroup, a cluster was left to a few waves: 6000 of
// 20 000 particles in a sphere of 1.5 took 108 ms, 2e5 in one of 20 14 ms.
constexpr int kRdfSlices = 64;

__global__ __launch_bounds__(kRdfThreads) void k_rdf(RdfArgs a)
{
    extern __shared__ unsigned long long h[];   // [nbins]
    __shared__ PairTables tabs[kRdfWaves];
    __shared__ double4 home[kRdfWaves][kRdfHomes];
    __shared__ double queue[kRdfWaves][128];
    __shared__ uint8_t pidx[kRdfWaves][kPieceTab];
    for (int b = threadIdx.x; b < a.nbins; b += kRdfThreads) h[b] = 0ull;
    __syncthreads();
    const int lane = threadIdx.x & 63;
    const int wv = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    int queued = 0;   // uniform
    auto pair = [&](int q, int first, int step, int end) {
        rdf_pair(a, q, first, step, end, tabs[wv], home[wv], queue[wv], pidx[wv], h, queued);
    };
    const int half = (a.g.nc[0] + 1) >> 1, pairs = a.g.nc[2] * a.g.nc[1] * half;
    const int blocks = (int)gridDim.x, waves = blocks * kRdfWaves;
    // neighbouring pairs to a workgroup (they share most of their rows) where a wave has one
    // at most (N = 2e4: 49 us a histogram with its build, 51 apart), else far apart
    const bool apart = pairs > waves;
    for (int q = (int)blockIdx.x * (apart ? 1 : kRdfWaves) + wv * (apart ? blocks : 1); q < pairs; q += waves)
        pair(q, 0, 1, a.own);
    const int slices = min(kRdfSlices, waves), shares = waves / slices, columns = (pairs + 63) / 64;
    const int wave = (int)blockIdx.x * kRdfWaves + wv;
    int turn = wave % slices;   // this wave's place in the deal of its share's passes, less what is dealt (mod slices)
    for (int col = wave / slices; col < columns && wave < shares * slices; col += shares) {
        const int q = lane * columns + col;
        int left = 0;
        if (q < pairs) {
            const int row = q / half, x0 = 2 * (q - row * half), x1 = min(x0 + 1, a.g.nc[0] - 1);
            const int32_t *start = a.cell_start + row * a.g.nc[0];
            left = max(0, (start[x1 + 1] - start[x0] + kRdfHomes - 1) / kRdfHomes - a.own);
        }
        for (uint64_t m = __builtin_amdgcn_ballot_w64(left > 0); m != 0; m &= m - 1) {   // uniform
            const int l = (int)__builtin_ctzll(m);
            pair(l * columns + col, a.own + turn, slices, 0x7fffffff);
            turn -= __builtin_amdgcn_readlane(left, l) % slices;
            if (turn < 0) turn += slices;
        }
    }
    wave_lds_fence();
    rdf_count(a, queue[wv], queued, h);
    __syncthreads();
    for (int b = threadIdx.x; b < a.nbins; b += kRdfThreads)
        if (h[b]) atomicAdd(&a.hist[b], h[b]);
}

// ---------------------------------------------------------------------------
// displacement tracking, MSD and VACF
// ---------------------------------------------------------------------------

struct TrackBox {
    double L[3], inv_L[3];
};

__global__ __launch_bounds__(kBlock) void k_track(int64_t N, TrackBox b, const double *__restrict__ x,
                                                  double *__restrict__ x_last, double *__restrict__ disp)
{
    const int64_t k = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (k >= 3 * N) return;
    const int a = (int)(k / N);   // the axis of component k (SoA [3][N])
    const double xn = x[k];
    double d = xn - x_last[k];
    d = d - b.L[a] * rint(d * b.inv_L[a]);
    disp[k] += d;
    x_last[k] = xn;
}

constexpr int kMsdBlocks = 1024;   // fixed grid: partials summed in one order whatever N is

// per-block partial sums of |disp|^2 and v0 . v over a fixed grid-stride
// assignment of particles, then one block adds the partials in block order
__global__ __launch_bounds__(kBlock) void k_msd_part(int64_t N, const double *__restrict__ disp,
                                                     const double *__restrict__ v0, const double *__restrict__ v,
                                                     double2 *__restrict__ part)
{
    __shared__ double red[kBlock];
    double m = 0.0, c = 0.0;
    for (int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x; i < N; i += (int64_t)kMsdBlocks * kBlock)
        for (int d = 0; d < 3; ++d) {
            const double u = disp[d * N + i];
            m = fma(u, u, m);
            c = fma(v0[d * N + i], v[d * N + i], c);
        }
    m = block_sum_256(m, red);
    __syncthreads();
    c = block_sum_256(c, red);
    if (threadIdx.x == 0) part[blockIdx.x] = make_double2(m, c);
}

__global__ __launch_bounds__(kBlock) void k_msd_final(int64_t N, const double2 *__restrict__ part,
                                                      double *__restrict__ out)
{
    __shared__ double red[kBlock];
    double m = 0.0, c = 0.0;
    for (int b = threadIdx.x; b < kMsdBlocks; b += kBlock) {
        m += part[b].x;
        c += part[b].y;
    }
    m = block_sum_256(m, red);
    __syncthreads();
    c = block_sum_256(c, red);
    if (threadIdx.x == 0) {
        out[0] = m / (double)N;
        out[1] = c / (double)N;
    }
}

}  // namespace
}  // namespace rbsog

using namespace rbsog;

extern "C" int rbsog_track_box(int64_t N, double Lx, double Ly, double Lz, const double *x_dev, double *x_last_dev,
                               double *disp_dev, void *hip_stream)
{
    if (N < 1 || N > ((int64_t)1 << 27) - 1) return fail(RBSOG_EINVAL, "N must lie in [1, 2^27 - 1]");
    const double Lb[3] = {Lx, Ly, Lz};
    TrackBox b{};
    for (int a = 0; a < 3; ++a) {
        if (!(Lb[a] > 0.0) || !std::isfinite(Lb[a])) return fail(RBSOG_EINVAL, "box edges must be positive and finite");
        b.L[a] = Lb[a];
        b.inv_L[a] = 1.0 / Lb[a];
    }
    if (!x_dev || !x_last_dev || !disp_dev) return fail(RBSOG_EINVAL, "null x, x_last or disp");
    const int64_t n3 = 3 * N;
    hipLaunchKernelGGL(k_track, dim3((unsigned)((n3 + kBlock - 1) / kBlock)), dim3(kBlock), 0, (hipStream_t)hip_stream,
                       N, b, x_dev, x_last_dev, disp_dev);
    HIPCHECK(hipGetLastError());
    return RBSOG_OK;
}

extern "C" int rbsog_track(int64_t N, double L, const double *x_dev, double *x_last_dev, double *disp_dev,
                           void *hip_stream)
{
    if (!(L > 0.0) || !std::isfinite(L)) return fail(RBSOG_EINVAL, "L must be positive and finite");
    return rbsog_track_box(N, L, L, L, x_dev, x_last_dev, disp_dev, hip_stream);
}

extern "C" int rbsog_msd_scratch_size(size_t *bytes)
{
    if (!bytes) return fail(RBSOG_EINVAL, "null bytes");
    *bytes = sizeof(double2) * kMsdBlocks;
    return RBSOG_OK;
}

extern "C" int rbsog_msd_vacf(int64_t N, const double *disp_dev, const double *v0_dev, const double *v_dev,
                              void *scratch_dev, size_t scratch_bytes, void *hip_stream, double *out_dev)
{
    if (N < 1 || N > ((int64_t)1 << 27) - 1) return fail(RBSOG_EINVAL, "N must lie in [1, 2^27 - 1]");
    if (!disp_dev || !v0_dev || !v_dev || !scratch_dev || !out_dev)
        return fail(RBSOG_EINVAL, "null disp, v0, v, scratch or out");
    if (scratch_bytes < sizeof(double2) * kMsdBlocks)
        return fail(RBSOG_EWORKSPACE, "scratch of %zu bytes is below the %zu needed", scratch_bytes,
                    sizeof(double2) * kMsdBlocks);
    hipStream_t st = (hipStream_t)hip_stream;
    hipLaunchKernelGGL(k_msd_part, dim3(kMsdBlocks), dim3(kBlock), 0, st, N, disp_dev, v0_dev, v_dev,
                       (double2 *)scratch_dev);
    HIPCHECK(hipGetLastError());
    hipLaunchKernelGGL(k_msd_final, dim3(1), dim3(kBlock), 0, st, N, (const double2 *)scratch_dev, out_dev);
    HIPCHECK(hipGetLastError());
    return RBSOG_OK;
}

extern "C" int rbsog_ssf_scratch_size(int64_t N, int m_s, size_t *bytes)
{
    if (!bytes) return fail(RBSOG_EINVAL, "null bytes");
    if (N < 1 || N > ((int64_t)1 << 27) - 1) return fail(RBSOG_EINVAL, "N must lie in [1, 2^27 - 1]");
    if (m_s < 1 || m_s > kMaxLatticeM) return fail(RBSOG_EINVAL, "m_s must lie in [1, %d]", kMaxLatticeM);
    *bytes = ssf_plan(N, m_s).total;
    return RBSOG_OK;
}

extern "C" int rbsog_ssf(int64_t N, double L, const double *x_dev, const double *w_dev, int m_s, void *scratch_dev,
                         size_t scratch_bytes, void *hip_stream, double *s_dev)
{
    size_t need = 0;
    int rc = rbsog_ssf_scratch_size(N, m_s, &need);
    if (rc) return rc;
    if (!(L > 0.0) || !std::isfinite(L)) return fail(RBSOG_EINVAL, "L must be positive and finite");
    if (!x_dev || !w_dev || !s_dev || !scratch_dev) return fail(RBSOG_EINVAL, "null x, w, s or scratch");
    if (((uintptr_t)scratch_dev % kAlign) != 0) return fail(RBSOG_EINVAL, "scratch must be 256-byte aligned");
    if (scratch_bytes < need) return fail(RBSOG_EWORKSPACE, "scratch of %zu bytes is below the %zu needed", scratch_bytes, need);
    const SsfPlan pl = ssf_plan(N, m_s);
    hipStream_t st = (hipStream_t)hip_stream;
    char *s = (char *)scratch_dev;
    // modes of the shells in (|n|^2, nx, ny, nz) order, unit weight, and the
    // first mode of each shell
    std::vector<int32_t> packed((size_t)pl.K);
    lattice_copy(m_s, packed.data());
    std::vector<double> modes(4 * (size_t)pl.K);
    std::vector<int64_t> start((size_t)m_s + 2, 0);
    for (int64_t i = 0; i < pl.K; ++i) {
        const uint32_t pk = (uint32_t)packed[(size_t)i];
        const int nx = (int)(pk & 1023u) - kLatticeBias, ny = (int)((pk >> 10) & 1023u) - kLatticeBias;
        const int nz = (int)((pk >> 20) & 1023u) - kLatticeBias;
        modes[4 * i] = nx;
        modes[4 * i + 1] = ny;
        modes[4 * i + 2] = nz;
        modes[4 * i + 3] = 1.0;
        start[(size_t)(nx * nx + ny * ny + nz * nz) + 1] += 1;
    }
    for (int m = 1; m <= m_s + 1; ++m) start[(size_t)m] += start[(size_t)m - 1];
    HIPCHECK(hipMemcpyAsync(s + pl.o_tab, phase_table(), sizeof(double) * 2 * kPhaseTable, hipMemcpyHostToDevice, st));
    if (pl.K > 0)
        HIPCHECK(hipMemcpyAsync(s + pl.o_modes, modes.data(), sizeof(double) * modes.size(), hipMemcpyHostToDevice, st));
    HIPCHECK(hipMemcpyAsync(s + pl.o_start, start.data(), sizeof(int64_t) * start.size(), hipMemcpyHostToDevice, st));
    const double4 *dm = (const double4 *)(s + pl.o_modes);
    double2 *drho = (double2 *)(s + pl.o_rho);
    for (int64_t c0 = 0; c0 < pl.K; c0 += pl.pass) {
        RhoArgs a{};
        a.N = (int)N;
        a.P = (int)std::min<int64_t>(pl.pass, pl.K - c0);
        a.chunk = pl.pass == pl.P ? rho_chunk((int)N, a.P) : pl.chunk;
        // a short last pass: a workgroup of few modes stages more groups, so smaller
        // ones (the partials fit: below 86 modes of groups that fill the staging area,
        // under N + P of them, where a full pass has 4 N)
        while ((255 / a.P + 2) * a.chunk > kRhoStage) a.chunk /= 2;
        a.nchunk = (int)((N + a.chunk - 1) / a.chunk);
        a.inv_L[0] = a.inv_L[1] = a.inv_L[2] = 1.0 / L;
        a.x = x_dev;
        a.q = w_dev;
        a.samp = dm + c0;
        a.part = (double2 *)(s + pl.o_part);
        a.rho = drho + c0;
        a.mixed = 0;
        a.tab = (const double2 *)(s + pl.o_tab);
        a.ss = make_sincos_short();
        HIPCHECK(launch_rho_partial(a, st));
        HIPCHECK(launch_rho_reduce(a, st));
    }
    hipLaunchKernelGGL(k_ssf_shells, dim3((m_s + kBlock / 64) / (kBlock / 64)), dim3(kBlock), 0, st, drho,
                       (const int64_t *)(s + pl.o_start), m_s, s_dev);
    HIPCHECK(hipGetLastError());
    HIPCHECK(hipStreamSynchronize(st));   // the host-side mode tables are released on return
    return RBSOG_OK;
}

extern "C" int rbsog_rdf(rbsog_handle *h, const double *x_dev, double r_max, int nbins, unsigned long long *hist_dev)
{
    if (!h || !x_dev || !hist_dev) return fail(RBSOG_EINVAL, "null handle, x or hist");
    if (!(r_max > 0.0) || !(r_max <= h->sog.r_c)) return fail(RBSOG_EINVAL, "r_max must lie in (0, r_c]");
    if (nbins < 1 || nbins > kRdfMaxBins) return fail(RBSOG_EINVAL, "nbins must lie in [1, %d]", kRdfMaxBins);
    // the positions into cell order on the fine grid (cells >= r_c / 2 >= r_max / 2)
    PermArgs in = perm_args(h, (double *)x_dev, nullptr, nullptr);
    HIPCHECK(launch_state_in(in, h->st));
    CellArgs ca = cell_args(h, h->gf, nullptr, false);
    HIPCHECK(launch_cell_build(ca, h->st));
    h->lists_valid = false;   // the rows moved: the next evaluation builds its lists again
    RdfArgs a{};
    a.nbins = nbins;
    a.g = h->gf;
    for (int d = 0; d < 3; ++d) a.w[d] = h->d.Lb[d] / (double)a.g.nc[d];
    a.xs = h->xs;
    a.cell_start = h->cell_start;
    a.rmax2 = r_max * r_max;
    a.dr = r_max / nbins;
    a.hist = hist_dev;
    for (int d = 0; d < 3; ++d)
        if (a.g.nc[d] < 6) return fail(RBSOG_EINVAL, "fine grid of %d cells is below the 6-cell window", a.g.nc[d]);
    const int pairs = a.g.nc[2] * a.g.nc[1] * ((a.g.nc[0] + 1) / 2);
    // home particles of a pair at uniform density, and four deviations of their number
    const double mean = 2.0 * (double)h->p.N / (double)a.g.ncell;
    a.own = (int)std::ceil((mean + 4.0 * std::sqrt(mean)) / kRdfHomes);
    hipLaunchKernelGGL(k_rdf, dim3(std::min(kRdfBlocks, (pairs + kRdfWaves - 1) / kRdfWaves)), dim3(kRdfThreads),
                       sizeof(unsigned long long) * (size_t)nbins, h->st, a);
    HIPCHECK(hipGetLastError());
    return RBSOG_OK;
}
