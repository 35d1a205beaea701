// gfx950 kernels of librbsog: far field, force assembly, second half-kick, energies.
#include <hip/hip_runtime.h>

#include "dev_common.h"

namespace rbsog {

// ---------------------------------------------------------------------------
// far field of the random batch (eq. UF):
//   f_i += -q_i (2 pi / L) sum_l coef_l n_l Im(exp(-i k_l . r_i) rho_l).
// A workgroup owns 64 consecutive particles (cell order), or 128 (PPL particles
// per lane), and has W waves with C chains each; chain c of wave g takes the
// samples l = g + W c mod W C of each LDS tile of 256 samples, so every particle's
// sum is spread over W lanes.  The partial sums are added in a fixed order, then
// near + far is written (in cell order, and/or in the caller's order) and the
// second half-kick applied in cell order; in a run of steps the next step's first
// half-kick and drift follow at once.  Two particles per lane share the LDS reads
// of a mode (bound beside the arithmetic otherwise) and give each wave two
// independent chains more, with W C = 4; a system whose workgroups would then
// fill the chip less than a few times over keeps one, and W C = 16 instead: its
// waves are few, and more waves or more chains in each hide more of what an
// instruction waits (N = 10 007, P = 193, mixed, a step with a thermostat: 29.9 ->
// 28.9 us; N = 6e4, P = 500, mixed: 86 -> 85; N = 2e5, P = 300, FP64: 195.6 -> 194.9).
//
// Bound by its vector instructions, 20 per (particle, mode) in FP64: three FMAs of
// the phase (which start from the mode's offset), 13 of the cosine, three to
// accumulate.  The table form (sine and cosine from a 1024-entry rotation table,
// then their product with rho) took 26 and two more LDS reads: N = 1e6, P = 500,
// 416 us against 323 (1.6e12 (particle, mode) terms a second).  Its error is the
// smaller one (18 systems of 900 to 1500 particles, RMS of the force against extended
// precision: 6.9e-16, 11.4e-16 with the table), because positions enter less whole
// revolutions, which halves what the phase's FMAs round.  FP64 matrix
// instructions do not help: the phases as a 16 x 16 x 4 product (72 cycles for 256
// terms) and the accumulation as 4 x 4 x 4 products (18 cycles for 64) hold up
// the FP64 vector unit for as long as the FMAs they replace.
// ---------------------------------------------------------------------------

constexpr int kFarTile = 256;
constexpr int kFarThreads = 256;   // the ensemble's workgroups

// A tile's samples in LDS: k = (n, phase offset) and w = -size n (FP64), or k =
// (n, coef) and w.xy = coef rho (mixed).
struct FarTile {
    double4 k[kFarTile];
    double2 w[kFarTile];
    double wz[kFarTile];
};

// Adds one mode to a particle's sum; s is r/L (FP64: less whole revolutions), so that
// n.s is the phase in revolutions.
template <bool MIXED>
__device__ inline void far_add(const FarArgs &a, const double4 &k, const double2 &w, double wz, const double s[3],
                               double acc[3])
{
    if (MIXED) {
        const double u = k.x * s[0] + k.y * s[1] + k.z * s[2];
        float sn, cs;
        sincos_rev_f32(u, &sn, &cs);
        const double im = w.y * (double)cs - w.x * (double)sn;
        acc[0] += im * k.x;
        acc[1] += im * k.y;
        acc[2] += im * k.z;
    } else {
        const double c = neg_cos_rev(fma(k.x, s[0], fma(k.y, s[1], fma(k.z, s[2], k.w))), a.ss);
        acc[0] = fma(c, w.x, acc[0]);
        acc[1] = fma(c, w.y, acc[1]);
        acc[2] = fma(c, wz, acc[2]);
    }
}

// A particle's row of what the far field adds to and moves.
struct FarRow {
    double fn[3], v[3], xb[3], m;
    int order;
};
template <bool DRIFT>
__device__ inline FarRow far_row(const FarArgs &a, int p)
{
    static_assert(kNearLanes == 1, "one partial near force per particle");
    FarRow r{};
#pragma unroll
    for (int d = 0; d < 3; ++d) r.fn[d] = a.fnear[(size_t)d * a.N + p];
    if (a.vs) {
#pragma unroll
        for (int d = 0; d < 3; ++d) {
            r.v[d] = a.vs[(size_t)d * a.N + p];
            if (DRIFT) r.xb[d] = a.xb[(size_t)d * a.N + p];
        }
        r.m = a.ms[p];
    }
    if (a.f || a.f_near_out || (DRIFT && a.th.on)) r.order = a.order[p];
    return r;
}

template <bool MIXED, bool DRIFT, int PPL, int W, int C>
__device__ inline void far_body(const FarArgs &a, int b)
{
    static_assert((W == 8 && C == 2) || (W == 4 && (C == 4 || C == 1)), "the orders of addition below");
    constexpr int G = W * C;   // mode groups: wave g's chain c takes the modes l = g + W c mod G
    constexpr int kPart = 64 * W * PPL;
    constexpr size_t kLds = sizeof(FarTile) > 3 * kPart * sizeof(double) ? sizeof(FarTile) : 3 * kPart * sizeof(double);
    __shared__ __align__(16) char lds[kLds];   // a tile of samples, then the waves' partials
    FarTile &tile = *(FarTile *)lds;
    double(*part)[kPart] = (double(*)[kPart])lds;
    const int t = threadIdx.x;
    const int g = __builtin_amdgcn_readfirstlane(t >> 6), lane = t & 63;   // g is uniform per wave
    if (a.gate_clear && b == 0 && t == 0) {
        if (a.rebuilds && *a.gate_clear) *a.rebuilds += 1;
        *a.gate_clear = 0;
    }
    double s[PPL][3], acc[C][PPL][3];
#pragma unroll
    for (int i = 0; i < PPL; ++i) {
        const int p = (b * PPL + i) * 64 + lane;
        const double4 pi = p < a.N ? a.xs[p] : make_double4(0.0, 0.0, 0.0, 0.0);
        if (MIXED) {
            s[i][0] = pi.x * a.inv_L[0];
            s[i][1] = pi.y * a.inv_L[1];
            s[i][2] = pi.z * a.inv_L[2];
        } else {
            s[i][0] = less_turns(pi.x, a.inv_L[0]);
            s[i][1] = less_turns(pi.y, a.inv_L[1]);
            s[i][2] = less_turns(pi.z, a.inv_L[2]);
        }
#pragma unroll
        for (int c = 0; c < C; ++c) acc[c][i][0] = acc[c][i][1] = acc[c][i][2] = 0.0;
    }
    // what the finishing wave reads besides the partials: in a small system it is
    // on its way while the modes are summed (its registers cost a larger one more)
    constexpr bool EARLY = W > 4;
    const int p = b * PPL * 64 + t;
    double4 pi{};
    FarRow row{};
    if (EARLY && g == 0 && p < a.N) {
        pi = a.xs[p];
        row = far_row<DRIFT>(a, p);
    }
    // chain c adds mode m of the tile to the wave's particles
    auto add = [&](int c, int m) {
        const double4 k0 = tile.k[m];
        const double2 w0 = tile.w[m];
        const double z0 = MIXED ? 0.0 : tile.wz[m];
#pragma unroll
        for (int i = 0; i < PPL; ++i) far_add<MIXED>(a, k0, w0, z0, s[i], acc[c][i]);
    };
    for (int l0 = 0; l0 < a.P; l0 += kFarTile) {
        __syncthreads();
        if (t < kFarTile && l0 + t < a.P) {
            const double4 k = a.samp[l0 + t];
            const double2 gk = a.gk[l0 + t];
            if (MIXED) {
                tile.k[t] = k;
                tile.w[t] = gk;
            } else {
                tile.k[t] = make_double4(k.x, k.y, k.z, gk.y);
                tile.w[t] = make_double2(-gk.x * k.x, -gk.x * k.y);
                tile.wz[t] = -gk.x * k.z;
            }
        }
        __syncthreads();
        int nl = min(kFarTile, a.P - l0);
        int m = g;
        if constexpr (C == 1) {
            // two modes per pass (independent chains), added in mode order
            for (; m + W < nl; m += 2 * W) {
                const double4 k0 = tile.k[m], k1 = tile.k[m + W];
                const double2 w0 = tile.w[m], w1 = tile.w[m + W];
                const double z0 = MIXED ? 0.0 : tile.wz[m], z1 = MIXED ? 0.0 : tile.wz[m + W];
#pragma unroll
                for (int i = 0; i < PPL; ++i) {
                    far_add<MIXED>(a, k0, w0, z0, s[i], acc[0][i]);
                    far_add<MIXED>(a, k1, w1, z1, s[i], acc[0][i]);
                }
            }
            if (m < nl) add(0, m);
        } else {
            for (; m + W * (C - 1) < nl; m += G) {
#pragma unroll
                for (int c = 0; c < C; ++c) add(c, m + W * c);
            }
#pragma unroll
            for (int c = 0; c < C - 1; ++c)
                if (m + W * c < nl) add(c, m + W * c);
        }
    }
    __syncthreads();   // the sample tile is done with: it holds the partials next
#pragma unroll
    for (int i = 0; i < PPL; ++i) {
        const int at = (g * PPL + i) * 64 + lane;   // wave g's partial of particle (i, lane)
#pragma unroll
        for (int d = 0; d < 3; ++d) {
            if constexpr (C == 1) part[d][at] = acc[0][i][d];
            else if constexpr (C == 2) part[d][at] = acc[0][i][d] + acc[1][i][d];
            else part[d][at] = (acc[0][i][d] + acc[2][i][d]) + (acc[1][i][d] + acc[3][i][d]);
        }
    }
    __syncthreads();
    if (t >= 64 * PPL) return;   // whole waves; thread t finishes particle t
    double ke = 0.0;
    if (p < a.N) {
        if (!EARLY) {
            pi = a.xs[p];
            row = far_row<DRIFT>(a, p);
        }
        double bx = 0.0, by = 0.0, bz = 0.0;
        // of 16 groups, (k + k8) + (k4 + k12) for k = 0 .. 3, then these four: the same
        // order whether eight waves or four held them
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            double sx = part[0][k * 64 * PPL + t], sy = part[1][k * 64 * PPL + t], sz = part[2][k * 64 * PPL + t];
            if constexpr (W == 8) {
                sx += part[0][(k + 4) * 64 * PPL + t];
                sy += part[1][(k + 4) * 64 * PPL + t];
                sz += part[2][(k + 4) * 64 * PPL + t];
            }
            bx += sx;
            by += sy;
            bz += sz;
        }
        const double scx = -pi.w * a.two_pi_over_L[0], scy = -pi.w * a.two_pi_over_L[1];
        const double scz = -pi.w * a.two_pi_over_L[2];
        const double fnx = row.fn[0], fny = row.fn[1], fnz = row.fn[2];
        double fx = fnx + scx * bx, fy = fny + scy * by, fz = fnz + scz * bz;
        if (a.fs) {
            a.fs[p] = fx;
            a.fs[a.N + p] = fy;
            a.fs[2 * a.N + p] = fz;
        }
        if (a.f || a.f_near_out) {
            const int i = row.order;
            if (a.f) {
                a.f[i] = fx;
                a.f[a.N + i] = fy;
                a.f[2 * a.N + i] = fz;
            }
            if (a.f_near_out) {
                a.f_near_out[i] = fnx;
                a.f_near_out[a.N + i] = fny;
                a.f_near_out[2 * a.N + i] = fnz;
            }
        }
        raise_any(a.flag, !isfinite(fx + fy + fz));
        if (a.vs) {
            double mi = row.m;
            double hm = a.half_dt / mi;
            double vx = row.v[0] + hm * fx, vy = row.v[1] + hm * fy, vz = row.v[2] + hm * fz;
            ke = 0.5 * mi * (vx * vx + vy * vy + vz * vz);
            if (DRIFT) {   // the next step's first half-kick and drift
                double x[3] = {pi.x, pi.y, pi.z}, v[3] = {vx, vy, vz};
                const double f[3] = {fx, fy, fz};
                bool bad = false;
                double d2 = kick_drift_row(x, v, f, hm, a.dt, a.L, a.inv_L, row.xb, 1, 0, &bad, a.th,
                                           (uint64_t)row.order, mi);
                vx = v[0];
                vy = v[1];
                vz = v[2];
                a.xs_next[p] = make_double4(x[0], x[1], x[2], pi.w);
                raise_any(a.flag, bad);
                raise_gate(a.gate_raise, d2, a.half_skin2, p);
            }
            a.vs[p] = vx;
            a.vs[a.N + p] = vy;
            a.vs[2 * a.N + p] = vz;
        }
    }
    if (a.kepart) {   // one partial per 64 particles: a fixed tree over the wave
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) ke += __shfl_down(ke, off);
        if (lane == 0 && b * PPL + g < far_blocks(a.N)) a.kepart[b * PPL + g] = ke;
    }
}

template <bool MIXED, bool DRIFT, int PPL, int W, int C>
__global__ __launch_bounds__(64 * W) void k_far(FarArgs a)
{
    far_body<MIXED, DRIFT, PPL, W, C>(a, (int)blockIdx.x);
}

template <bool MIXED>
__global__ __launch_bounds__(kFarThreads) void k_far_batch(const FarArgs *__restrict__ tab,
                                                           const EnsItem *__restrict__ items, uint64_t *advance)
{
    const EnsItem e = items[blockIdx.x];
    if (advance && blockIdx.x == 0 && threadIdx.x == 0) *advance += 1;
    const FarArgs &a = tab[e.r];
    // the order of the system alone
    if (a.N < kFarPairN) far_body<MIXED, false, 1, 4, 4>(a, e.b);
    else far_body<MIXED, false, 1, 4, 1>(a, e.b);
}

hipError_t launch_far_batch(const FarArgs *tab, const EnsItem *items, int n, bool mixed, uint64_t *advance,
                            hipStream_t st)
{
    if (!tab || !items || n < 1) return hipErrorInvalidValue;
    if (mixed) hipLaunchKernelGGL(k_far_batch<true>, dim3(n), dim3(kFarThreads), 0, st, tab, items, advance);
    else hipLaunchKernelGGL(k_far_batch<false>, dim3(n), dim3(kFarThreads), 0, st, tab, items, advance);
    return hipGetLastError();
}

template <bool MIXED, bool DRIFT>
static void launch_far_as(const FarArgs &a, hipStream_t st)
{
    const int nb = far_blocks(a.N);
    if (a.N >= kFarPairN) hipLaunchKernelGGL((k_far<MIXED, DRIFT, 2, 4, 1>), dim3((nb + 1) / 2), dim3(256), 0, st, a);
    else if (a.N >= kFarWideN) hipLaunchKernelGGL((k_far<MIXED, DRIFT, 1, 4, 4>), dim3(nb), dim3(256), 0, st, a);
    else hipLaunchKernelGGL((k_far<MIXED, DRIFT, 1, 8, 2>), dim3(nb), dim3(512), 0, st, a);
}

hipError_t launch_far(const FarArgs &a, hipStream_t st)
{
    if (a.N < 1 || a.P < 1 || !a.xs || !a.order || !a.samp || !a.gk || !a.fnear || (!a.f && !a.fs) || !a.flag ||
        (a.vs && (!a.ms || !a.kepart)) || (a.drift && (!a.vs || !a.xb || !a.xs_next || !a.gate_raise)))
        return hipErrorInvalidValue;
    if (a.drift) {
        if (a.mixed) launch_far_as<true, true>(a, st);
        else launch_far_as<false, true>(a, st);
    } else {
        if (a.mixed) launch_far_as<true, false>(a, st);
        else launch_far_as<false, false>(a, st);
    }
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// energies: fixed-order sums of the block partials
// ---------------------------------------------------------------------------

// One workgroup per row: a step leaves the partials of its row in a set of its
// own, and one launch adds up to kEnergyRows rows: a workgroup alone takes 5 us
// at N = 1000 and took 48 at N = 1e6 (bound by the latency of its loads, eight
// of which are now in flight), sixteen of them take as long as one.  row: the
// set, and the row of `out` after the first `shift` (the ensemble writes row
// shift + row0).
__device__ inline void energy_body(const EnergyArgs &a, int row, uint64_t shift)
{
    __shared__ double red[kBlock];
    const double *epart = a.epart + (size_t)row * 2 * a.nnear;
    double un = strided_sum(epart, a.nnear), wn = strided_sum(epart + a.nnear, a.nnear);
    double uf = strided_sum(a.eF + (size_t)row * a.P, a.P), wf = strided_sum(a.eW + (size_t)row * a.P, a.P);
    double ke = a.kepart ? strided_sum(a.kepart + (size_t)row * a.nfar, a.nfar) : 0.0;
    un = block_sum_256(un, red);
    __syncthreads();
    uf = block_sum_256(uf, red);
    __syncthreads();
    ke = block_sum_256(ke, red);
    __syncthreads();
    wn = block_sum_256(wn, red);
    __syncthreads();
    wf = block_sum_256(wf, red);
    if (threadIdx.x == 0) {
        double *o = a.out + kEnergyCols * (shift + a.row0 + (uint64_t)row);
        o[0] = un;
        o[1] = uf;
        o[2] = a.Uk0;
        o[3] = a.Uself;
        o[4] = a.Ubg;
        o[5] = a.ke_set ? a.ke_set[row] : ke;
        o[6] = wn;
        o[7] = wf;
    }
}

__global__ __launch_bounds__(kBlock) void k_energy(EnergyArgs a)
{
    energy_body(a, (int)blockIdx.x, 0);
}

__global__ __launch_bounds__(kBlock) void k_energy_batch(const EnergyArgs *__restrict__ tab,
                                                         const EnsItem *__restrict__ items, const uint64_t *shift)
{
    energy_body(tab[items[blockIdx.x].r], 0, *shift - 1);   // the far field has moved the counter on
}

hipError_t launch_energy_batch(const EnergyArgs *tab, const EnsItem *items, int n, const uint64_t *shift,
                               hipStream_t st)
{
    if (!tab || !items || n < 1 || !shift) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_energy_batch, dim3(n), dim3(kBlock), 0, st, tab, items, shift);
    return hipGetLastError();
}

hipError_t launch_energy(const EnergyArgs &a, hipStream_t st)
{
    if (!a.epart || !a.eF || !a.eW || !a.out || a.rows < 1 || a.rows > kEnergyRows) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_energy, dim3(a.rows), dim3(kBlock), 0, st, a);
    return hipGetLastError();
}


}  // namespace rbsog
