// Device helpers shared by the kernels of librbsog.
#pragma once

#include <hip/hip_runtime.h>

#include "dev_math.h"
#include "launch.h"

namespace rbsog {

// Cell coordinate of a position: clamp(floor(x nc / L), 0, nc - 1); a NaN maps to 0.
__device__ inline int cell_coord(double x, double inv_cell, int nc)
{
    double f = floor(x * inv_cell);
    if (!(f >= 0.0)) return 0;
    if (f >= (double)(nc - 1)) return nc - 1;
    return (int)f;
}

// Raises *flag when cond holds in any active lane of the wave: one atomic per
// wave (the lowest such lane), not one per lane.  Every lane of a step may
// raise the same rebuild gate (a hot system with no skin), and same-address
// atomics from every lane serialise in the L2.
__device__ inline void raise_any(int32_t *flag, bool cond)
{
    const uint64_t m = __ballot(cond);
    if (m != 0 && (int)(threadIdx.x & 63) == __ffsll((unsigned long long)m) - 1) atomicOr(flag, 1);
}

// Raises a rebuild gate when some particle of the wave has moved more than half
// the skin since the last build (d2: its squared displacement).  With no skin
// any motion leaves the lists stale, so the gate is raised by the system's
// first particle alone: one atomic per launch instead of one per wave (at 1e6
// particles the 15 625 same-address atomics of the waves serialise for
// ~0.15 ms).
__device__ inline void raise_gate(int32_t *gate, double d2, double half_skin2, int p)
{
    raise_any(gate, half_skin2 > 0.0 ? !(d2 <= half_skin2) : p == 0);
}

// Fixed-order sum over a 256-thread block; valid in thread 0.
__device__ inline double block_sum_256(double v, double *red)
{
    int t = threadIdx.x;
    red[t] = v;
    __syncthreads();
#pragma unroll
    for (int off = 128; off > 0; off >>= 1) {
        if (t < off) red[t] += red[t + off];
        __syncthreads();
    }
    return red[0];
}

// A thread's share of the sum of v[0 .. n) over a kBlock-thread workgroup (added
// in index order), eight loads in flight.
__device__ inline double strided_sum(const double *v, int n)
{
    double s = 0.0;
    int b = threadIdx.x;
    for (; b + 7 * kBlock < n; b += 8 * kBlock) {
        double u[8];
#pragma unroll
        for (int k = 0; k < 8; ++k) u[k] = v[b + k * kBlock];
#pragma unroll
        for (int k = 0; k < 8; ++k) s += u[k];
    }
    for (; b < n; b += kBlock) s += v[b];
    return s;
}

// The thermostat's three normal deviates of particle i (caller index) for the
// drift into force index `step`: four uniforms ((w >> 11) + 1) 2^-53 in (0, 1]
// from Philox4x64-10(counter (i, step, 1, 0), key (seed, replica)) -- word 2 =
// 1 keeps them apart from the mode draws -- through the Box-Muller transform.
__device__ inline void langevin_normals(uint64_t i, const Thermo &th, double z[3])
{
    uint64_t w[4];
    philox4x64_10(i, th.step, 1, 0, th.seed, (uint64_t)th.replica, w);
    double u[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) u[k] = (double)((w[k] >> 11) + 1) * 0x1p-53;
    const double twopi = 6.283185307179586;
    const double r0 = sqrt(-2.0 * log(u[0])), r1 = sqrt(-2.0 * log(u[2]));
    z[0] = r0 * cos(twopi * u[1]);
    z[1] = r0 * sin(twopi * u[1]);
    z[2] = r1 * cos(twopi * u[3]);
}

// First half-kick and drift of one particle (cell position p): v += hm f,
// x += dt v, wrapped into [0, L); returns the squared minimum-image distance
// from the build position xb and sets *bad on a step of a box length or more.
// The drift kernel and the far kernel's fused form both run this, so that
// their trajectories agree bit for bit.  hm = dt / (2 m); with a thermostat
// on, ci is the particle's caller index and m its mass.
__device__ inline double kick_drift_row(double x[3], double v[3], const double f[3], double hm, double dt,
                                        const double Lb[3], const double inv_Lb[3], const double *xb, int N, int p,
                                        bool *bad, const Thermo &th, uint64_t ci, double m)
{
    double d2 = 0.0;
    double z[3] = {0.0, 0.0, 0.0}, sig = 0.0;
    if (th.on) {
        langevin_normals(ci, th, z);
        sig = sqrt(th.c2kT / m);
    }
#pragma unroll
    for (int d = 0; d < 3; ++d) {
        double vv = v[d] + hm * f[d];
        double dx;
        if (th.on) {   // half drift, Ornstein-Uhlenbeck update, half drift
            const double v2 = th.c1 * vv + sig * z[d];
            dx = 0.5 * dt * vv + 0.5 * dt * v2;
            vv = v2;
        } else {
            dx = dt * vv;
        }
        const double L = Lb[d];
        *bad |= !(fabs(dx) < L);
        double xx = x[d] + dx;
        if (xx >= L) xx -= L;
        if (xx < 0.0) xx += L;
        if (xx >= L) xx = 0.0;
        v[d] = vv;
        x[d] = xx;
        double s = xx - xb[d * N + p];
        s = fma(-L, rint(s * inv_Lb[d]), s);
        d2 = fma(s, s, d2);
    }
    return d2;
}

// First half-kick and drift of workgroup b's rows; raises the rebuild gate of
// this step and clears the next one's (when the caller alternates two).
__device__ inline void kick_drift_body(const KickDriftArgs &a, int b)
{
    int p = b * kBlock + threadIdx.x;
    if (p == 0 && a.gate_next) *a.gate_next = 0;
    if (p >= a.N) return;
    const double hm = (0.5 * a.dt) / a.ms[p];
    const double4 r = a.xs[p];
    double x[3] = {r.x, r.y, r.z};
    double v[3] = {a.vs[p], a.vs[a.N + p], a.vs[2 * a.N + p]};
    if (a.vscale) {   // a global bath's half-steps since the last kick
        const double sc = *a.vscale;
        v[0] = v[0] * sc;
        v[1] = v[1] * sc;
        v[2] = v[2] * sc;
    }
    const double f[3] = {a.fs[p], a.fs[a.N + p], a.fs[2 * a.N + p]};
    bool bad = false;
    double d2 = kick_drift_row(x, v, f, hm, a.dt, a.L, a.inv_L, a.xb, a.N, p, &bad, a.th,
                               a.th.on ? (uint64_t)a.order[p] : 0, a.ms[p]);
    for (int d = 0; d < 3; ++d) a.vs[d * a.N + p] = v[d];
    a.xs[p] = make_double4(x[0], x[1], x[2], r.w);
    raise_any(a.flag, bad);
    raise_gate(a.gate, d2, a.half_skin2, p);
}

// ---------------------------------------------------------------------------
// structure factors.  Particles are cut into groups of C (the "chunk") and the
// lanes of the grid are laid out flat over (group s, sample l), lane s P + l,
// so every lane of every wave has work whatever P is.  A workgroup stages the
// particles of the groups its lanes touch in LDS; each lane sums its group in
// two interleaved streams and writes one partial per (group, sample); a second
// kernel adds the partials of each sample in a fixed order.
// ---------------------------------------------------------------------------

// x inv_L less whole revolutions, in one rounding: n times it is the phase less whole
// revolutions, with half the rounding of n (x inv_L) and of the sums over the axes.
__device__ inline double less_turns(double x, double inv_L) { return fma(x, inv_L, -rint(x * inv_L)); }

// One particle's term q exp(i k.r) of a mode; k.p is the phase in the unit that the
// precision's sine and cosine take: revolutions (mixed) or 1/T of them (FP64, T the
// entries of the rotation table: kPhaseTab, or kFarTab with FINE).  UNIT (FP64): exp(i k.r) alone, the rotation
// by the table entry accumulated as it is formed (the caller multiplies the sum
// by the charge all its particles have): two instructions fewer of 20.  Its large
// parts go to re, im and its small ones (with the rotation's sine, at most pi/T) to
// re1, im1, re - re1 and im + im1 being the term: one rounding a term at the size of
// the sum, as where the rotated values are formed first, not two.  Bound by its
// instructions: 262 147 particles and 500 modes take 93 us, where the loop over charges
// and pairs of particles took 105.
template <bool MIXED, bool FINE = false, bool UNIT = false>
__device__ inline void rho_term(const RhoArgs &a, const double2 *tab, const double4 &k, const double4 &p,
                                double &re, double &im, double *re1 = nullptr, double *im1 = nullptr)
{
    static_assert(!(MIXED && UNIT), "the mixed terms take the charge");
    double u = k.x * p.x + k.y * p.y + k.z * p.z;
    if (MIXED) {
        float sn, cs;
        sincos_rev_f32(u, &sn, &cs);
        re = fma(p.w, (double)cs, re);
        im = fma(p.w, (double)sn, im);
    } else if (UNIT) {
        double2 t;
        double sp, cp;
        if (FINE) rotation_far(u, tab, a.sf, &t, &sp, &cp);
        else rotation_tab(u, tab, a.ss, &t, &sp, &cp);
        re = fma(t.y, cp, re);
        im = fma(t.x, cp, im);
        *re1 = fma(t.x, sp, *re1);
        *im1 = fma(t.y, sp, *im1);
    } else {
        double sn, cs;
        if (FINE) sincos_rev_far(u, tab, a.sf, &sn, &cs);
        else sincos_rev_tab(u, tab, a.ss, &sn, &cs);
        re = fma(p.w, cs, re);
        im = fma(p.w, sn, im);
    }
}

// Sum over the n staged particles sp[0..n) of a mode, in two interleaved
// chains (n uniform over the workgroup: four particles per pass, so that the
// loop's own instructions are shared by four terms).
template <bool MIXED, bool FINE, bool UNIT>
__device__ inline double2 rho_group(const RhoArgs &a, const double2 *tab, const double4 &k, const double4 *sp, int n)
{
    double re0 = 0.0, im0 = 0.0, re1 = 0.0, im1 = 0.0, rs = 0.0, is = 0.0;
    int i = 0;
    for (; i + 3 < n; i += 4) {
        rho_term<MIXED, FINE, UNIT>(a, tab, k, sp[i], re0, im0, &rs, &is);
        rho_term<MIXED, FINE, UNIT>(a, tab, k, sp[i + 1], re1, im1, &rs, &is);
        rho_term<MIXED, FINE, UNIT>(a, tab, k, sp[i + 2], re0, im0, &rs, &is);
        rho_term<MIXED, FINE, UNIT>(a, tab, k, sp[i + 3], re1, im1, &rs, &is);
    }
    for (; i < n; ++i) rho_term<MIXED, FINE, UNIT>(a, tab, k, sp[i], re0, im0, &rs, &is);
    return UNIT ? make_double2(re0 + re1 - rs, im0 + im1 + is) : make_double2(re0 + re1, im0 + im1);
}

// groups of fewer particles are summed with their charges: asking whether these are
// all equal takes longer than it saves
constexpr int kUnitChunk = 64;

template <bool CELL, bool MIXED, bool FINE>
__device__ inline void rho_partial_body(const RhoArgs &a, int b)
{
    // dynamic LDS: the rotation table (FP64), then the staged particles
    constexpr int T = FINE ? kFarTab : kPhaseTab;
    extern __shared__ double4 lds[];
    double2 *tab = (double2 *)lds;
    double4 *sp = lds + (MIXED ? 0 : T / 2);
    const int t = threadIdx.x;
    const int64_t g0 = (int64_t)b * kBlock;
    const int s_lo = (int)(g0 / a.P);
    const int s_hi = (int)min((int64_t)a.nchunk - 1, (g0 + kBlock - 1) / a.P);
    const int j_lo = s_lo * a.chunk;
    const int j_hi = min(a.N, (s_hi + 1) * a.chunk);
    // every particle of the workgroup with one charge (a one-component plasma):
    // the sums run without it
    const bool ask = !MIXED && a.chunk >= kUnitChunk;   // uniform over the launch
    const double q0 = !ask ? 0.0 : CELL ? a.xs[j_lo].w : a.q[j_lo];
    bool other = false;
    for (int k = t; k < j_hi - j_lo; k += kBlock) {
        int j = j_lo + k;
        double4 v;
        if (CELL) v = a.xs[j];
        else v = make_double4(a.x[j], a.x[a.N + j], a.x[2 * a.N + j], a.q[j]);
        if (!MIXED) other |= !(v.w == q0);
        double x = v.x * a.inv_L[0], y = v.y * a.inv_L[1], z = v.z * a.inv_L[2];
        if (!MIXED) {
            x = less_turns(v.x, a.inv_L[0]);
            y = less_turns(v.y, a.inv_L[1]);
            z = less_turns(v.z, a.inv_L[2]);
        }
        sp[k] = make_double4(x, y, z, v.w);
    }
    if (!MIXED) {
        const double2 *src = FINE ? a.tab_fine : a.tab;
        for (int k = t; k < T; k += kBlock) tab[k] = src[k];
    }
    bool unit = false;   // uniform
    if (ask) unit = !__syncthreads_or(other);
    else __syncthreads();
    const int64_t g = g0 + t;
    if (g >= (int64_t)a.nchunk * a.P) return;
    const int s = (int)(g / a.P), l = (int)(g - (int64_t)s * a.P);
    double4 k = a.samp[l];
    if (!MIXED) {   // the phase in the table's steps
        k.x *= T;
        k.y *= T;
        k.z *= T;
    }
    const double4 *group = sp + (s * a.chunk - j_lo);
    // whole groups but in the workgroup that holds the last one
    const int n = (s_hi + 1) * a.chunk <= a.N ? a.chunk : min(a.N, (s + 1) * a.chunk) - s * a.chunk;
    if (unit) {
        if constexpr (!MIXED) {
            const double2 r = rho_group<false, FINE, true>(a, tab, k, group, n);
            a.part[g] = make_double2(q0 * r.x, q0 * r.y);
        }
    } else {
        a.part[g] = rho_group<MIXED, FINE, false>(a, tab, k, group, n);
    }
}

// k^2 G / Fhat of a mode (G = -dFhat/d(k^2)): from the table by |n|^2 in a
// cube, from the Fourier coefficients in a cuboid.
__device__ inline double mode_vm(const RhoArgs &a, const double4 &sl)
{
    if (a.vm) {   // |n|^2 from the mode's integer components (exact in FP64)
        const int m = (int)(sl.x * sl.x + sl.y * sl.y + sl.z * sl.z);
        return a.vm[m];
    }
    const double tp = 6.283185307179586;
    const double kx = tp * sl.x * a.inv_L[0], ky = tp * sl.y * a.inv_L[1], kz = tp * sl.z * a.inv_L[2];
    const double k2 = kx * kx + ky * ky + kz * kz;
    double F = 0.0, G = 0.0;
    for (int g = 0; g < a.nG; ++g) {
        const double e = exp(-a.fb[g] * k2);
        F += a.fa[g] * e;
        G += a.fa[g] * a.fb[g] * e;
    }
    return F > 0.0 ? k2 * G / F : 0.0;
}

// What the far field takes of a mode's weight cf and structure factor: cf rho
// (mixed), or its size and the phase offset with which Im(exp(-i k.r) cf rho) =
// size cos(2 pi (k.r/(2 pi) + offset)), offset = 1/4 - arg(rho)/(2 pi) (FP64).  The
// angle is taken from the nearest axis and quarter turns are added to it: every
// particle's phase carries the offset's error, 1.6e-17 revolutions RMS (3.6e-17 with
// an angle of up to pi, rounded before it is scaled).
__device__ inline double2 far_coef(int mixed, double cf, double re, double im)
{
    if (mixed) return make_double2(cf * re, cf * im);
    const bool swap = fabs(im) > fabs(re);   // nearer to the imaginary axis
    const double x = swap ? im : re, y = swap ? re : im;
    const double phi = atan2(x < 0.0 ? -y : y, fabs(x));   // within pi/4
    const double base = swap ? (x < 0.0 ? 0.5 : 0.0) : (x < 0.0 ? -0.25 : 0.25);
    return make_double2(cf * sqrt(re * re + im * im), fma(swap ? phi : -phi, 0.15915494309189535, base));
}

// Fixed-order sum of the chunk partials, one workgroup per kRedModes adjacent
// samples so that each partial row is read as one contiguous segment.  Thread
// t takes sample l = kRedModes b + (t mod kRedModes) and adds the partials of
// groups c, c + 64, c + 128, ... (c = t / kRedModes, four loads in flight); the
// 16 threads of a wave that share a sample are added by a fixed butterfly and
// the four waves in order.
__device__ inline void rho_reduce_body(const RhoArgs &a, int b)
{
    constexpr int kLanes = kBlock / kRedModes;   // group streams per sample
    __shared__ double2 red[kBlock / 64][kRedModes];
    const int t = threadIdx.x, m = t % kRedModes, c0 = t / kRedModes;
    const int l = b * kRedModes + m;
    const bool live = l < a.P;
    const double2 *col = a.part + (live ? l : 0);
    const size_t P = (size_t)a.P;
    const int nch = live ? a.nchunk : 0;
    // what the finishing threads need besides is on its way with the partials, and
    // the last of those all together: at small sizes the launch is a chain of
    // loads that wait for one another (N = 10 007, P = 193, mixed: a step 30.4 ->
    // 29.9 us; N = 60 000, P = 500: 87 -> 86)
    const bool last = t < kRedModes && live;
    double4 sl{};
    if (last) sl = a.samp[l];
    double re = 0.0, im = 0.0;
    int c = c0;
    for (; c + 3 * kLanes < nch; c += 4 * kLanes) {
        double2 v0 = col[(size_t)c * P], v1 = col[(size_t)(c + kLanes) * P];
        double2 v2 = col[(size_t)(c + 2 * kLanes) * P], v3 = col[(size_t)(c + 3 * kLanes) * P];
        re += v0.x;
        im += v0.y;
        re += v1.x;
        im += v1.y;
        re += v2.x;
        im += v2.y;
        re += v3.x;
        im += v3.y;
    }
    double2 v[3];   // up to three more, all in flight
#pragma unroll
    for (int k = 0; k < 3; ++k) v[k] = c + k * kLanes < nch ? col[(size_t)(c + k * kLanes) * P] : double2{0.0, 0.0};
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        re += v[k].x;   // + 0 past the last group
        im += v[k].y;
    }
    const double vm = last && a.eW ? mode_vm(a, sl) : 0.0;
#pragma unroll
    for (int off = 32; off >= kRedModes; off >>= 1) {
        re += __shfl_xor(re, off);
        im += __shfl_xor(im, off);
    }
    if ((t & 63) < kRedModes) red[t >> 6][m] = make_double2(re, im);
    __syncthreads();
    if (last) {
        re = 0.0;
        im = 0.0;
#pragma unroll
        for (int w = 0; w < kBlock / 64; ++w) {
            re += red[w][t].x;
            im += red[w][t].y;
        }
        const double cf = sl.w;
        a.rho[l] = make_double2(re, im);
        if (a.gk) {   // a step's modes: the far field's coefficients and the energies
            a.gk[l] = far_coef(a.mixed, cf, re, im);
            a.eF[l] = 0.5 * cf * (re * re + im * im);
        }
        if (a.eW) a.eW[l] = cf * (re * re + im * im) * (1.5 - vm);
        if (a.rho_out) {
            a.rho_out[2 * l] = re;
            a.rho_out[2 * l + 1] = im;
        }
    }
}

}  // namespace rbsog
