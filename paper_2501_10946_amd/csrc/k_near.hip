// gfx950 kernel of librbsog: the near field of eq. (3.8),
//   f_i = sum_{j : |d| < r_c} q_i q_j [F_N1(r) + F_N2(r)] d,   d = r_i - r_j (minimum image),
//   F_N1 = exp(-r/lambda)(1 + r/lambda)/r^3,  F_N2 = -2 sum_g c_g s_g exp(-s_g r^2),
//   (F_N1 summed over the terms a_t exp(-r/l_t)(1 + r/l_t)/r^3 of a two-term kernel),
// and the near energy U_N = 1/2 sum q_i q_j (Y(r) - F(r)).
//
// The cell grid is the fine one, cells of width w = L / floor(2L / (r_c + skin))
// >= (r_c + skin) / 2, so the neighbour stencil is 5 x 5 x 5 cells; cell order
// makes each x-row of 5 cells one contiguous index range (two where it wraps
// around the box).
//
//   k_nlist  a wave lists the particles of two x-adjacent cells: lanes take
//            the candidates of the pair's 5 x 5 x 6-cell window 64 at a time
//            (loads coalesced along the rows) and test each against every
//            home particle in turn; the accepted ones are appended in lane
//            order straight into the particles' lists, in window order, with
//            a count per particle;
//   k_near   a wave evaluates the lists of 16 consecutive particles, four
//            lanes each: lane s takes entries s, s + 4, ... two at a time, with
//            the rows of the next two and the indices of the two after in
//            flight, and the four add their sums before three of them store the
//            force.  In FP64 the pair function is, when its fit is accurate, one polynomial
//            in r (r^3 times the force factor, 24 to 28 FMAs, no exponential),
//            otherwise the number of Gaussians is a template parameter for
//            the common counts; coefficients stay in scalar registers.  When a
//            particle's list overflowed at the build, its lanes walk the
//            candidates of the current positions, plane by plane.  A
//            single system's launch also computes the structure-factor
//            partial sums in some of its workgroups: the gathers above leave
//            the arithmetic units idle part of the time, the partial sums
//            keep them busy (the reduction follows as a launch of its own).
//
// Why four lanes side by side: a gather instruction looks its rows up one cache
// line after the other, so what it costs is the number of lines its 64 lanes
// touch (random rows of 32 bytes: 111 cycles of a compute unit for 64 rows,
// runs of four consecutive rows: 60).  Consecutive entries of one list are
// often consecutive rows; the earlier split (three lanes per particle in three
// different waves) had none of that, wrote and read three partial forces per
// particle, and a wave waited for the longest of 64 lists where it now waits
// for the longest of 16.  Of 4, 8 and 16 lanes, 4 is the fastest (N = 1e5: 82
// us a step, 8: 87, 16: 98; the earlier split: 87).
//
// Lists hold every j within r_c + skin at the build.  The step path rebuilds
// them (and the cell order) only when some particle has moved more than
// skin / 2 since the last build, so every pair within r_c is listed; pairs
// listed but now beyond r_c are skipped in the evaluation.
//
// Each lane sums its share of a particle's force in list order and the
// shares are added in a fixed order: the result is deterministic.
#include <hip/hip_runtime.h>

#include "dev_common.h"
#include "dev_window.h"

namespace rbsog {

constexpr int kNearPlanes = 5;                 // stencil planes dz = -2..2
constexpr int kListThreads = 64 * kListWaves;  // list build: one cell pair per wave
constexpr int kShiftBits = 5;                  // image-shift code 0..26 in the top bits of a range start
constexpr uint32_t kIndexMask = (1u << (32 - kShiftBits)) - 1u;

// The argument block where it lies in memory (the kernel's argument segment, or
// the ensemble's table): its fields are scalar loads.  near_args_again makes
// the compiler load them anew from there on, instead of keeping every field of
// the block in scalar registers from the kernel's start: the pair polynomials
// need those, and what does not fit is kept in lanes of vector registers and
// read back with an instruction each.
typedef const __attribute__((address_space(4))) NearArgs NearMem;
typedef const double __attribute__((address_space(4))) *ScalarMem;

__device__ inline NearMem &near_args_again(NearMem &a)
{
    NearMem *p = &a;
    __asm__ volatile("" : "+s"(p));
    return *p;
}


// Distance from coordinate y to the slab [c w - m, (c + 1) w + m] (0 inside).
__device__ inline double slab_gap(double y, int c, double w, double m)
{
    double lo = (double)c * w - m, hi = (double)(c + 1) * w + m;
    return fmax(0.0, fmax(lo - y, y - hi));
}

// One candidate range: particles [start, end) of the cell-ordered copy, all
// under one image shift (code = xc + 3 yc + 9 zc, each 0/1/2 for -L/0/+L).
struct Range {
    int32_t start_code;     // start | code << 27
    int32_t end;
};

// The (particle, plane) a lane works on, with its home cell.
struct Lane {
    int p, plane;
    double4 pi;
    int cx, cy, cz, zc;     // home x, y; wrapped z cell of the plane and its shift code
    double gz;              // z-gap from the particle to the plane
};

__device__ inline Lane make_lane(NearMem &a, int p, int plane)
{
    Lane l;
    l.p = p;
    l.plane = plane;
    l.pi = make_double4(0.0, 0.0, 0.0, 0.0);
    l.cx = l.cy = l.cz = 0;
    l.zc = 1;
    l.gz = 1e300;
    if (p < a.N) {
        const int nfz = a.g.nc[2];
        l.pi = a.xs[p];
        l.cx = cell_coord(l.pi.x, a.g.inv_cell[0], a.g.nc[0]);
        l.cy = cell_coord(l.pi.y, a.g.inv_cell[1], a.g.nc[1]);
        int czu = cell_coord(l.pi.z, a.g.inv_cell[2], nfz) + plane - 2;
        l.gz = slab_gap(l.pi.z, czu, a.w[2], a.margin);
        l.cz = czu;
        if (czu < 0) { l.cz += nfz; l.zc = 0; } else if (czu >= nfz) { l.cz -= nfz; l.zc = 2; }
    }
    return l;
}

// The candidate ranges of row `row` (dy = row - 2) for a lane within radius
// sqrt(R2) (R2 <= the list radius squared, which the fine grid is built for):
// 0, 1 or 2 ranges.
__device__ inline int row_ranges(NearMem &a, const Lane &l, int row, double R2, Range out[2])
{
    const int nf = a.g.nc[0], nfy = a.g.nc[1];
    const double m = a.margin;
    int cyu = l.cy + row - 2;
    double gy = slab_gap(l.pi.y, cyu, a.w[1], m);
    double rem = R2 - gy * gy - l.gz * l.gz;
    if (!(rem > 0.0)) return 0;
    int dxlo = -2, dxhi = 2;
    for (int k = 0; k < 2; ++k) {   // at most two x-cells per side can be culled
        double gl = slab_gap(l.pi.x, l.cx + dxlo, a.w[0], m);
        if (dxlo < 0 && !(gl * gl < rem)) ++dxlo;
        double gh = slab_gap(l.pi.x, l.cx + dxhi, a.w[0], m);
        if (dxhi > 0 && !(gh * gh < rem)) --dxhi;
    }
    int xa = l.cx + dxlo, xb = l.cx + dxhi;   // unwrapped; xb - xa <= 4 < nf
    int cyw = cyu, yc = 1;
    if (cyw < 0) { cyw += nfy; yc = 0; } else if (cyw >= nfy) { cyw -= nfy; yc = 2; }
    int base = (l.cz * nfy + cyw) * nf;
    int code = 3 * yc + 9 * l.zc;
    int n = 0;
    // piece left of the wrap (or the whole row), then the piece past it
    int lo0 = xa < 0 ? xa + nf : xa, hi0 = xa < 0 ? nf - 1 : min(xb, nf - 1);
    int xc0 = xa < 0 ? 0 : 1;
    int s0 = a.cell_start[base + lo0], e0 = a.cell_start[base + hi0 + 1];
    // (out[] written at fixed indices only, so that it stays in registers)
    if (s0 < e0) {
        out[0] = Range{(int32_t)((uint32_t)s0 | ((uint32_t)(code + xc0) << 27)), e0};
        n = 1;
    }
    if (xa < 0 || xb > nf - 1) {
        int hi1 = xa < 0 ? xb : xb - nf;
        int xc1 = xa < 0 ? 1 : 2;
        int s1 = a.cell_start[base], e1 = a.cell_start[base + hi1 + 1];
        if (s1 < e1) {
            const Range r{(int32_t)((uint32_t)s1 | ((uint32_t)(code + xc1) << 27)), e1};
            if (n == 0) out[0] = r;
            else out[1] = r;
            ++n;
        }
    }
    return n;
}

// FP64 1/sqrt(x) for x > 0: the hardware estimate (measured within 2^-24.2 of
// it over [1, 4)) and one third-order step, y (1 + e/2 + 3 e^2/8) with e = 1 -
// x y^2, whose remainder 5 e^3/16 is below 2^-70: five instructions where two
// second-order steps take seven.
__device__ inline double rsqrt_f64(double x)
{
    const double y = __builtin_amdgcn_rsq(x);
    const double e = fma(-(x * y), y, 1.0);
    return fma(y * e, fma(0.375, e, 0.5), y);
}

// Gaussians of the pair function: NG > 0 is a compile-time count, 0 the
// run-time count of the argument block; NG < 0: the whole pair function from
// the polynomials of the argument block, of degree -NG (FP64).  kPolyNG, the
// full degree, also serves polynomials of a lower degree (their higher powers
// are zero, and Horner's first steps then leave the leading coefficient
// unchanged, so the result is the same bit for bit).
constexpr int kPolyNG = -28;
template <int NG>
__device__ inline int gauss_count(NearMem &a) { return NG > 0 ? NG : a.sog.n; }

// Horner in y of the degree-D polynomial c (ascending powers).
template <int D>
__device__ inline double near_poly_eval(ScalarMem c, double y)
{
    static_assert(D >= 1 && D <= 28, "the argument block holds 29 powers");
    double p = c[D];
#pragma unroll
    for (int k = D - 1; k >= 0; --k) p = fma(p, y, c[k]);
    return p;
}

// A launch with energies needs two polynomials' coefficients, more than the
// scalar registers hold: the force polynomial stays in them, the energy
// polynomial's come from the scalar cache at each pass over two pairs.
// p0, p1 = the degree-D polynomial c at y0, y1.
template <int D>
__device__ inline void near_poly_pair(ScalarMem c, double y0, double y1, double &p0, double &p1)
{
    __asm__ volatile("" : "+s"(c));   // loaded here, not kept from an earlier pass
    p0 = c[D];
    p1 = c[D];
#pragma unroll
    for (int k = D - 1; k >= 0; --k) {
        const double ck = c[k];
        p0 = fma(p0, y0, ck);
        p1 = fma(p1, y1, ck);
    }
}

// The sums of a lane over its pairs: force, energy and virial per unit charge of
// the particle itself, whose own charge multiplies them once at the end.
struct NearSums {
    double fx, fy, fz, en, vir;
};

// A pair's displacement, squared distance, force factor and energy per unit
// charge of the particle, from the raw difference of the positions and the
// neighbour's charge.  Evaluated whatever r2 is (a pair beyond r_c or a
// stand-in entry gives values nobody adds), so that the terms of several pairs
// interleave; near_add adds those of a pair that counts.
struct PairTerms {
    double dx, dy, dz, r2, fac, u;
    double y, qir;   // the energy polynomial's argument and factor (near_energy)
};

// IMG: the axes (bit d for axis d) on which the minimum-image step is taken;
// the callers leave an axis out only where the step provably changes nothing
// (near_image_axes).
template <bool MIXED, bool ENERGY, int NG, int IMG>
__device__ inline PairTerms pair_terms(NearMem &a, double dx, double dy, double dz, double qj)
{
    PairTerms t;
    // d by the minimum image (|d| < r_c <= L_d/3)
    if (IMG & 1) dx = fma(-a.g.L[0], rint(dx * a.inv_L[0]), dx);
    if (IMG & 2) dy = fma(-a.g.L[1], rint(dy * a.inv_L[1]), dy);
    if (IMG & 4) dz = fma(-a.g.L[2], rint(dz * a.inv_L[2]), dz);
    // written out as FMAs: the compiler's own contraction of a sum of squares
    // may pick another product to fuse depending on how d was formed, and the
    // IMG variants must give the same bits
    const double r2 = fma(dz, dz, fma(dy, dy, dx * dx));
    t.dx = dx;
    t.dy = dy;
    t.dz = dz;
    t.r2 = r2;
    t.u = 0.0;
    if (MIXED) {
        float r2f = (float)r2;
        float irf = __builtin_amdgcn_rsqf(r2f);
        float rf = r2f * irf;
        float ey = __builtin_amdgcn_exp2f(-rf * a.sog.f.inv_lambda_log2e);
        float f1 = ey * (1.0f + rf * a.sog.f.inv_lambda);
        if (a.sog.two) {   // the second Yukawa term of a two-term kernel
            const float ez = __builtin_amdgcn_exp2f(-rf * a.sog.f.inv_lambda2_log2e);
            f1 = fmaf(a.sog.f.ya2, ez * (1.0f + rf * a.sog.f.inv_lambda2), a.sog.f.ya1 * f1);
            ey = fmaf(a.sog.f.ya2, ez, a.sog.f.ya1 * ey);
        }
        f1 = f1 * (irf * irf * irf);
        float gs = 0.0f, fs = 0.0f;
#pragma unroll
        for (int g = 0; g < (NG < 0 ? 0 : gauss_count<NG>(a)); ++g) {
            float eg = __builtin_amdgcn_exp2f(-a.sog.f.s_log2e[g] * r2f);
            gs = fmaf(a.sog.f.cs2[g], eg, gs);
            if (ENERGY) fs = fmaf(a.sog.f.c[g], eg, fs);
        }
        t.fac = qj * (double)(f1 - gs);
        if (ENERGY) t.u = qj * (double)(ey * irf - fs);
    } else if constexpr (NG < 0) {
        // H(r) / r^3 and K(r) / r with H, K the polynomials in y = 2 r / r_c - 1
        double ir = rsqrt_f64(r2);
        double r = r2 * ir;
        const double y = fma(r, a.sog.y_scale, -1.0);
        t.fac = qj * (near_poly_eval<-NG>(a.sog.hpoly, y) * (ir * ir * ir));
        if (ENERGY) {
            t.y = y;
            t.qir = qj * ir;
        }
    } else {
        double ir = rsqrt_f64(r2);
        double r = r2 * ir;
        double ey = exp2_nonpos(-r * a.sog.inv_lambda_log2e, a.e2);
        double f1 = ey * fma(r, a.sog.inv_lambda, 1.0);
        if (a.sog.two) {   // the second Yukawa term of a two-term kernel
            const double ez = exp2_nonpos(-r * a.sog.inv_lambda2_log2e, a.e2);
            f1 = fma(a.sog.ya2, ez * fma(r, a.sog.inv_lambda2, 1.0), a.sog.ya1 * f1);
            ey = fma(a.sog.ya2, ez, a.sog.ya1 * ey);
        }
        f1 = f1 * (ir * ir * ir);
        double gs = 0.0, fs = 0.0;
        {
#pragma unroll
            for (int g = 0; g < gauss_count<NG>(a); ++g) {
                double eg = exp2_nonpos(-a.sog.s_log2e[g] * r2, a.e2);
                gs = fma(a.sog.cs2[g], eg, gs);
                if (ENERGY) fs = fma(a.sog.c[g], eg, fs);
            }
        }
        t.fac = qj * (f1 - gs);
        if (ENERGY) t.u = qj * (ey * ir - fs);
    }
    return t;
}

// The energies of two pairs whose pair function is a polynomial.
template <int NG>
__device__ inline void near_energy(ScalarMem kpoly, PairTerms &t0, PairTerms &t1)
{
    if constexpr (NG < 0) {
        double k0, k1;
        near_poly_pair<-NG>(kpoly, t0.y, t1.y, k0, k1);
        t0.u = t0.qir * k0;
        t1.u = t1.qir * k1;
    }
}

template <bool ENERGY>
__device__ inline void near_add(NearSums &s, const PairTerms &t)
{
    __asm__ volatile("");   // kept a branch: as selects the sums cost three times the instructions
    s.fx = fma(t.fac, t.dx, s.fx);
    s.fy = fma(t.fac, t.dy, s.fy);
    s.fz = fma(t.fac, t.dz, s.fz);
    if (ENERGY) {
        s.en += t.u;
        s.vir = fma(t.fac, t.r2, s.vir);   // d . F of the pair
    }
}

// ---------------------------------------------------------------------------
// neighbour lists
// ---------------------------------------------------------------------------

// One wave lists the neighbours of the home particles of cell pair q,
// kListHomes of them per pass over the window.  Lanes take 64 consecutive
// candidates of the window at a time (loads coalesced along the rows); each
// home particle of the pass, its position read from LDS by every lane (a
// broadcast), is tested against all 64, and the accepted ones are appended
// in lane order (ballot / mbcnt) to that particle's list.  So a particle's list holds
// the candidates within the list radius in window order — planes, rows, wrap
// pieces, cell order — the same list, entry for entry, as a walk of the
// particle's own 5 x 5 x 5 cells: the pair window's extra cells lie at least
// 2 w >= r_c + skin away from the other cell's particles.  A particle with
// more than list_rows(kp) neighbours gets the count list_rows(kp) + 1 (its
// lanes then walk the cells in the evaluation).
//
// Bound by the vector and scalar instructions of its tests (~10 candidates of
// 64 pass one): a test is three FMAs and a compare (|c|^2 - 2 h.c < R^2 -
// |h|^2) where the difference took seven instructions, and two homes share the
// loop control, since the four SIMDs of a compute unit share one scalar unit
// (with the running counts and the overflow check in scalar registers too, 19
// scalar instructions a test, the launch took 0.54 ms).  N = 1e6 plasma: 0.44
// -> 0.37 ms a build, 222 -> 169 M vector instructions.
constexpr int kListHomes = 16;

// The tests of homes hp and hp + 1 of a pass against a chunk of 64 candidates
// (one per lane: image-shifted position, its square, particle index j), and the
// appends: the accepted lanes as one wave mask (the test, less the home's own
// lane: own is the pass's home a lane holds), under which they store at positions by
// mbcnt from the list's running end.  Appends past the capacity all land on the
// row's last entry: the list is then marked overflowed and never read.  The
// homes' data are read from LDS (a broadcast), not held in registers for every
// home.  Two homes at a time: their LDS reads overlap, and the scalar unit,
// which the four SIMDs of a compute unit share, has half the loop control.
__device__ inline void nlist_test(const double4 *home, double px, double py, double pz, double pp, int j, int own,
                                  int32_t *pass_row, uint32_t rows, int hp, uint32_t *slot)
{
    __asm__ volatile("" ::: "memory");
    const double4 h0 = home[hp], h1 = home[hp + 1];
    const double t0 = fma(h0.x, px, fma(h0.y, py, fma(h0.z, pz, pp)));
    const double t1 = fma(h1.x, px, fma(h1.y, py, fma(h1.z, pz, pp)));
    const uint64_t m[2] = {__builtin_amdgcn_ballot_w64(t0 < h0.w) & __builtin_amdgcn_ballot_w64(own != hp),
                           __builtin_amdgcn_ballot_w64(t1 < h1.w) & __builtin_amdgcn_ballot_w64(own != hp + 1)};
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const uint32_t last = (uint32_t)(hp + i + 1) * rows - 1u;
        const uint32_t k = min(__builtin_amdgcn_mbcnt_hi((uint32_t)(m[i] >> 32),
                                                         __builtin_amdgcn_mbcnt_lo((uint32_t)m[i], slot[hp + i])), last);
        if (__builtin_amdgcn_inverse_ballot_w64(m[i])) *(int32_t *)((char *)pass_row + (k << 2)) = j;
        slot[hp + i] += (uint32_t)__popcll(m[i]);
    }
}

__device__ inline void nlist_pair(const NearArgs &a, int q, int wv)
{
    __shared__ PairTables tabs[kListWaves];
    __shared__ double4 home[kListWaves][kListHomes];
    __shared__ uint8_t pidx[kListWaves][kPieceTab];
    const int lane = threadIdx.x & 63;
    PairTables &w = tabs[wv];
    PairWindow win;
    double centre[3];
    if (!pair_window<true>(a.g, a.w, a.cell_start, q, w, centre, win)) return;   // uniform per wave
    const int total = win.total;
    const bool tabled = window_pieces(w, total, pidx[wv]);   // uniform
    const uint32_t rows = (uint32_t)list_rows(a.kp);
    // The home particles are consecutive candidates of the window's central
    // row (dy = dz = 0, no image shift): piece 24 of that row, or piece 25
    // when the row wraps at the low x side (its first piece is then the
    // wrapped cells).  home_c is the candidate index of h_beg, so the lane
    // that holds a home itself follows from the lane's candidate index.
    const int home_c = win.h_beg - __builtin_amdgcn_readfirstlane(w.first[pair_window_home_piece(a.g, q)]);
    // the list radius squared with a relative margin of 1e-12 and the rounding
    // of an image-shifted position (a few ulp of the box edge): a candidate is
    // tested in another form than the evaluation's difference, and a pair on
    // the radius must not be lost to the rounding (extra pairs beyond r_c are
    // skipped by the evaluation)
    const double Lmax = fmax(a.g.L[0], fmax(a.g.L[1], a.g.L[2]));
    const double R2 = a.rl2 * (1.0 + 1e-12) + 0x1p-48 * Lmax * sqrt(a.rl2);
    for (int hb = win.h_beg; hb < win.h_end; hb += kListHomes) {
        const int nh = min(kListHomes, win.h_end - hb);   // uniform
        if (lane < kListHomes) {   // |c - h|^2 < R2 as |c|^2 - 2 h.c < R2 - |h|^2; past nh nothing passes
            double4 h = make_double4(0.0, 0.0, 0.0, -HUGE_VAL);
            if (lane < nh) {
                const double4 r = a.xs[hb + lane];
                const double hx = r.x - centre[0], hy = r.y - centre[1], hz = r.z - centre[2];
                h = make_double4(-2.0 * hx, -2.0 * hy, -2.0 * hz, R2 - (hx * hx + hy * hy + hz * hz));
            }
            home[wv][lane] = h;
        }
        wave_lds_fence();
        // the pass's homes' lists are consecutive rows from pass_row on; slot[hh]
        // is the next entry of home hh counted from pass_row (hh rows + count;
        // a wave-uniform value held in a vector register, where mbcnt adds it)
        int32_t *pass_row = a.nbr + list_at(hb, 0, (int)rows);
        uint32_t slot[kListHomes];
#pragma unroll
        for (int hh = 0; hh < kListHomes; ++hh) {
            slot[hh] = (uint32_t)hh * rows;
            __asm__("" : "+v"(slot[hh]));
        }
        const int hc = home_c + (hb - win.h_beg);   // candidate index of the pass's first home
        for (int c0 = 0; c0 < total; c0 += 64) {
            const int c = c0 + lane;
            int j = -1;
            double px = 0.0, py = 0.0, pz = 0.0, pp = HUGE_VAL;   // the candidate, image-shifted; none past the last
            if (c < total) {
                const int l = tabled ? (int)pidx[wv][c] : window_piece(w.pref, c);
                j = w.first[l] + c;
                const double4 qj = a.xs[j];
                px = qj.x + w.shift[0][l];
                py = qj.y + w.shift[1][l];
                pz = qj.z + w.shift[2][l];
                pp = px * px + py * py + pz * pz;
            }
            const int own = c - hc;   // the pass's home whose own lane this is (any other value: none)
#pragma unroll
            for (int hp = 0; hp < kListHomes; hp += 2)
                if (hp < nh) nlist_test(home[wv], px, py, pz, pp, j, own, pass_row, rows, hp, slot);   // uniform
        }
        uint32_t mine = 0;
#pragma unroll
        for (int hh = 0; hh < kListHomes; ++hh)
            if (lane == hh) mine = slot[hh] - (uint32_t)hh * rows;
        if (lane < nh) {
            a.nbr_cnt[hb + lane] = (int)(mine > rows ? rows + 1u : mine);
            if (mine == 0) pass_row[(uint32_t)lane * rows] = hb + lane;   // entry 0 is always a valid index
        }
        // the positions of the next pass overwrite these
        wave_lds_fence();
    }
}

__device__ inline void nlist_body(const NearArgs &a, int lb)
{
    if (a.gate && *a.gate == 0) return;
    const int wv = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    nlist_pair(a, lb * kListWaves + wv, wv);
}

// ---------------------------------------------------------------------------
// evaluation
// ---------------------------------------------------------------------------

// The axes on which a pair of this wave may need the minimum image (bit d:
// axis d), uniform over the wave: those along which some home particle lies
// within r_c of a face (with a relative margin of 1e-6).  A home particle
// farther from both faces of an axis sees every particle within r_c of it at
// its own unwrapped coordinate on that axis, so the raw difference is the
// displacement itself and the minimum-image step would return it unchanged
// (rint of a ratio below 1/2 is 0); a farther particle shows a raw difference
// at least as large as its true one and stays beyond r_c either way.  Lanes
// past N count as interior.  1 for the x axis alone (a wave of cell-ordered
// particles crosses the box along x), 7 whenever y or z is needed.
__device__ inline int near_image_axes(NearMem &a, const double4 &pi, int p)
{
    const double m = sqrt(a.rc2) * (1.0 + 1e-6);
    const bool live = p < a.N;
    const bool ex = live && !(pi.x >= m && pi.x <= a.g.L[0] - m);
    const bool eyz = live && !(pi.y >= m && pi.y <= a.g.L[1] - m && pi.z >= m && pi.z <= a.g.L[2] - m);
    if (__builtin_amdgcn_ballot_w64(eyz)) return 7;
    return __builtin_amdgcn_ballot_w64(ex) ? 1 : 0;
}

// Row j of the cell-ordered positions by a 32-bit byte offset from the
// wave-uniform base (j < 2^27: the offset fits), one address operation
// fewer per neighbour than a 64-bit index.
__device__ inline double4 xs_row(NearMem &a, int j)
{
    return *(const double4 *)((const char *)a.xs + ((uint32_t)j << 5));
}

// A lane's share of particle p's list: lane `sub` of its kNearShare lanes takes
// entries sub, sub + kNearShare, ...; `steps` (uniform over the wave, at least
// 1) covers the longest list of the wave's particles.  Past the end of its
// particle's list a lane repeats the last entry (entry 0 is valid in an empty
// list too), which is not added.  Two entries per pass; the rows of the next
// two start loading into the same registers once the differences are formed,
// and the indices of the two after them follow.  row0 is the wave's first
// list, `at` this lane's first entry and `last` its particle's last, in bytes
// from there.
template <bool MIXED, bool ENERGY, int NG, int IMG>
__device__ inline void near_list(NearMem &args, const double4 &pi, const char *row0, uint32_t at, uint32_t last,
                                 int steps, NearSums &s)
{
    NearMem &a = near_args_again(args);
    constexpr uint32_t kStep = kNearShare * sizeof(int32_t);
    auto entry = [&](uint32_t b) { return *(const int32_t *)(row0 + min(b, last)); };
    double4 q0 = xs_row(a, entry(at)), q1 = xs_row(a, entry(at + kStep));
    int j0 = entry(at + 2 * kStep), j1 = entry(at + 3 * kStep);
    for (int k = 0; k < steps; k += 2) {   // uniform
        double dx0 = pi.x - q0.x, dy0 = pi.y - q0.y, dz0 = pi.z - q0.z, w0 = q0.w;
        double dx1 = pi.x - q1.x, dy1 = pi.y - q1.y, dz1 = pi.z - q1.z, w1 = q1.w;
        // the differences before the loads below: no copies of the rows
        __asm__ volatile("" : "+v"(dx0), "+v"(dy0), "+v"(dz0), "+v"(w0), "+v"(dx1), "+v"(dy1), "+v"(dz1), "+v"(w1)
                         :: "memory");
        q0 = xs_row(a, j0);
        q1 = xs_row(a, j1);
        j0 = entry(at + 4 * kStep);
        j1 = entry(at + 5 * kStep);
        PairTerms t0 = pair_terms<MIXED, ENERGY, NG, IMG>(a, dx0, dy0, dz0, w0);
        PairTerms t1 = pair_terms<MIXED, ENERGY, NG, IMG>(a, dx1, dy1, dz1, w1);
        // both evaluated before either is added under its mask: the two chains
        // interleave and share their scalar coefficients
        __asm__ volatile("" : "+v"(t0.fac), "+v"(t1.fac));
        if (ENERGY) {
            if (!MIXED) near_energy<NG>(a.sog.kpoly, t0, t1);
            __asm__ volatile("" : "+v"(t0.u), "+v"(t1.u));
        }
        if (at <= last && t0.r2 < a.rc2) near_add<ENERGY>(s, t0);
        if (at + kStep <= last && t1.r2 < a.rc2) near_add<ENERGY>(s, t1);
        at += 2 * kStep;
    }
}

// Sum over a particle's kNearShare lanes, in every one of them.
template <int CTRL>
__device__ inline double dpp_add(double v)
{
    const uint64_t u = (uint64_t)__double_as_longlong(v);
    const uint32_t lo = (uint32_t)__builtin_amdgcn_mov_dpp((int)(uint32_t)u, CTRL, 0xf, 0xf, true);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_mov_dpp((int)(u >> 32), CTRL, 0xf, 0xf, true);
    return v + __longlong_as_double((long long)(((uint64_t)hi << 32) | lo));
}

__device__ inline double share_sum(double v)
{
    v = dpp_add<0xB1>(v);   // quad_perm [1,0,3,2]
    v = dpp_add<0x4E>(v);   // quad_perm [2,3,0,1]
    return v;
}

// lb: the logical workgroup, kNearHomes consecutive particles of kNearShare lanes
// each.
// SPLIT: choose the minimum-image axes per wave (near_image_axes); the served
// ensemble's small replicas have nearly every wave at a face, so their batch
// launch takes every axis and saves the code.
template <bool MIXED, bool ENERGY, int NG, bool SPLIT = true>
__device__ inline void near_body(NearMem &a0, int lb)
{
    NearMem &a = near_args_again(a0);
    static_assert(kNearShare == 4, "share_sum adds 4 lanes");
    const int t = threadIdx.x, sub = t & (kNearShare - 1);
    const int rows = list_rows(a.kp);
    const int p = lb * kNearHomes + t / kNearShare;
    double4 pi = make_double4(0.0, 0.0, 0.0, 0.0);
    int total = 0;
    if (p < a.N) {
        pi = a.xs[p];
        total = a.nbr_cnt[p];
    }
    const bool walk = total > rows;   // the list overflowed at the build
    if (walk) total = 0;
    int longest = 0;   // of the wave's particles
#pragma unroll
    for (int k = 0; k < 64; k += kNearShare) longest = max(longest, __builtin_amdgcn_readlane(total, k));
    const int steps = (longest + kNearShare - 1) / kNearShare;
    NearSums s{};
    if (steps > 0) {   // uniform
        const int pw = min(__builtin_amdgcn_readfirstlane(p), a.N - 1);   // the wave's first particle
        const char *row0 = (const char *)(a.nbr + list_at(pw, 0, rows));
        const uint32_t mine = (uint32_t)((min(p, a.N - 1) - pw) * rows);   // entry 0 of this particle, from there
        // a particle without entries has none to add: its lanes start past entry 0
        const uint32_t at = 4u * (mine + (uint32_t)sub + (total ? 0u : 1u));
        const uint32_t last = 4u * (mine + (uint32_t)max(total - 1, 0));
        const int img = SPLIT ? near_image_axes(a, pi, p) : 7;
        if (img == 0) near_list<MIXED, ENERGY, NG, 0>(a, pi, row0, at, last, steps, s);
        else if (img == 1) near_list<MIXED, ENERGY, NG, 1>(a, pi, row0, at, last, steps, s);
        else near_list<MIXED, ENERGY, NG, 7>(a, pi, row0, at, last, steps, s);
    }
    if (walk) {
        // the particle's lanes walk the cells of the stencil around the
        // current position.  Particles may have moved up to skin/2 out of
        // the cells they were sorted into (and wrapped around the box), so
        // the cells are culled with the list radius and the pair function
        // itself (minimum image, r < r_c) decides.
#pragma unroll 1
        for (int plane = 0; plane < kNearPlanes; ++plane) {
            const Lane l = make_lane(a, p, plane);
            if (l.gz * l.gz < a.rl2) {
#pragma unroll 1
                for (int row = 0; row < 5; ++row) {
                    Range g[2];
                    const int n = row_ranges(a, l, row, a.rl2, g);
#pragma unroll
                    for (int k = 0; k < 2; ++k) {   // fixed indices: g stays in registers
                        if (k >= n) break;
                        const int j0 = g[k].start_code & (int32_t)kIndexMask;
                        for (int j = j0 + sub; j < g[k].end; j += kNearShare) {
                            if (j == p) continue;
                            const double4 q = a.xs[j];
                            PairTerms u =
                                pair_terms<MIXED, ENERGY, NG, 7>(a, pi.x - q.x, pi.y - q.y, pi.z - q.z, q.w);
                            if (ENERGY && !MIXED) near_energy<NG>(a.sog.kpoly, u, u);
                            if (u.r2 < a.rc2) near_add<ENERGY>(s, u);
                        }
                    }
                }
            }
        }
    }
    // the particle's lanes added in a fixed order; three of them store
    NearMem &o = near_args_again(a);
    const double fx = pi.w * share_sum(s.fx), fy = pi.w * share_sum(s.fy), fz = pi.w * share_sum(s.fz);
    if (p < o.N && sub < 3) o.fnear[(size_t)sub * o.N + p] = sub == 0 ? fx : sub == 1 ? fy : fz;
    if (ENERGY) {
        __shared__ double2 red[kNearThreads / 64];
        // each pair is seen from both ends: half of its energy and virial from each
        double e = share_sum(0.5 * pi.w * s.en), w = share_sum(0.5 * pi.w * s.vir);
#pragma unroll
        for (int off = kNearShare; off < 64; off <<= 1) {
            e += __shfl_xor(e, off);
            w += __shfl_xor(w, off);
        }
        if ((t & 63) == 0) red[t >> 6] = make_double2(e, w);
        __syncthreads();
        if (t == 0) {
            double es = 0.0, ws = 0.0;
#pragma unroll
            for (int k = 0; k < kNearThreads / 64; ++k) {
                es += red[k].x;
                ws += red[k].y;
            }
            o.epart[lb] = es;
            o.epart[near_blocks(o.N) + lb] = ws;
        }
    }
}

// Single system: workgroups remapped so that neighbouring groups share an XCD.
__global__ __launch_bounds__(kListThreads) void k_nlist(NearArgs a)
{
    nlist_body(a, xcd_block((int)blockIdx.x, (int)gridDim.x));
}

// Without energies: held to the registers of 5 waves per SIMD (the cell walk of
// an overflowed list alone would take more; the gathers want the waves).
template <bool MIXED, bool ENERGY, int NG>
__global__ __launch_bounds__(kNearThreads) __attribute__((amdgpu_waves_per_eu(!ENERGY ? 5 : 1))) void k_near(
    NearArgs a)
{
    static_assert(kNearThreads == kBlock, "the structure-factor workgroups have kBlock threads");
    const int b = (int)blockIdx.x;
    int rb = -1, nb = 0;   // a structure-factor workgroup, or a near one
    if (a.nrho == 0 || !a.interleave) {
        if (b < a.nrho) rb = b;
        else nb = b - a.nrho;
    } else {
        // The structure-factor workgroups are spread evenly through the launch in
        // whole groups of 8 (one per XCD), so that every compute unit holds
        // arithmetic-bound partial sums beside the near field's gather-bound
        // waves; the near groups keep their dispatch order, and with it the XCD
        // mapping, and the partial last group is a near group.
        const int64_t gr = a.nrho / 8, gn = (gridDim.x - a.nrho + 7) / 8, G = gr + gn;
        const int64_t g = b / 8;
        const int64_t before = (g * gr + G - 1) / G;          // structure-factor groups before group g
        const int64_t upto = ((g + 1) * gr + G - 1) / G;
        if (upto > before) rb = (int)(before * 8 + (b & 7));
        else nb = (int)((g - before) * 8 + (b & 7));
    }
    if (rb >= 0) {   // uniform per workgroup
        if (rb < rho_blocks(a.red.nchunk, a.red.P)) rho_partial_body<true, MIXED, true>(a.red, rb);
        return;
    }
    // the argument block is the kernel's only argument
    near_body<MIXED, ENERGY, NG>(*(NearMem *)__builtin_amdgcn_kernarg_segment_ptr(),
                                 xcd_block(nb, (int)gridDim.x - a.nrho));
}

__global__ __launch_bounds__(kListThreads) void k_nlist_batch(const NearArgs *__restrict__ tab,
                                                              const EnsItem *__restrict__ items)
{
    const EnsItem e = items[blockIdx.x];
    nlist_body(tab[e.r], e.b);
}

// Every replica of one kind, whatever its number of Gaussians or its polynomials'
// degree (a branch that is uniform over the workgroup), and their structure-factor
// partial sums (items with b < 0: workgroup ~b of the replica's partials).  One
// launch for each number of Gaussians and one for the partials leaves the chip
// half empty at the end of each: 16 replicas of 500 to 27 000 particles with five
// numbers of Gaussians in mixed precision took 71 us a step in six launches and
// take 38 in one.
template <NearKind KIND>
__global__ __launch_bounds__(kNearThreads) void k_near_batch(const NearArgs *__restrict__ tab,
                                                             const RhoArgs *__restrict__ rho,
                                                             const EnsItem *__restrict__ items)
{
    const EnsItem e = items[blockIdx.x];
    constexpr bool MIXED = KIND == NearKind::kMixed;
    if (e.b < 0) {   // uniform per workgroup
        rho_partial_body<true, MIXED, true>(rho[e.r], ~e.b);
        return;
    }
    NearMem &a = *(NearMem *)(uintptr_t)(tab + e.r);
    if constexpr (KIND == NearKind::kPoly) {
        if (a.sog.poly <= 24) near_body<false, true, -24, false>(a, e.b);
        else if (a.sog.poly <= 26) near_body<false, true, -26, false>(a, e.b);
        else near_body<false, true, kPolyNG, false>(a, e.b);
    } else {
        switch (a.sog.n) {
        case 1: near_body<MIXED, true, 1, false>(a, e.b); return;
        case 2: near_body<MIXED, true, 2, false>(a, e.b); return;
        case 3: near_body<MIXED, true, 3, false>(a, e.b); return;
        case 4: near_body<MIXED, true, 4, false>(a, e.b); return;
        case 5: near_body<MIXED, true, 5, false>(a, e.b); return;
        case 6: near_body<MIXED, true, 6, false>(a, e.b); return;
        case 7: near_body<MIXED, true, 7, false>(a, e.b); return;
        case 8: near_body<MIXED, true, 8, false>(a, e.b); return;
        default: near_body<MIXED, true, 0, false>(a, e.b); return;
        }
    }
}

// A launch with a missing buffer is refused on the host.
static bool near_args_ok(const NearArgs &a)
{
    return a.N >= 1 && a.xs && a.cell_start && a.nbr && a.nbr_cnt && a.fnear && a.kp >= 1 &&
           a.g.nc[0] >= 6 && a.g.nc[1] >= 6 && a.g.nc[2] >= 6 &&
           a.rc2 > 0.0 && a.rl2 >= a.rc2 && a.w[0] > 0.0 && a.w[1] > 0.0 && a.w[2] > 0.0 && (!a.energy || a.epart) && a.nrho >= 0 && a.nrho % 8 == 0 &&
           (a.nrho == 0 || (a.red.xs && rho_partial_ok(a.red) && a.red.mixed == a.mixed && (a.mixed || a.red.tab_fine) &&
                            a.nrho >= rho_blocks(a.red.nchunk, a.red.P)));
}

hipError_t launch_nlist(const NearArgs &a, hipStream_t st)
{
    if (!near_args_ok(a)) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_nlist, dim3(nlist_blocks(a.g.nc)), dim3(kListThreads), 0, st, a);
    return hipGetLastError();
}

template <bool MIXED, bool ENERGY>
static void launch_near_ng(const NearArgs &a, dim3 grid, hipStream_t st)
{
    dim3 block(kNearThreads);
    const size_t lds = a.nrho > 0 ? rho_lds_bytes(a.red.P, a.red.chunk, MIXED, true) : 0;
    if (!MIXED && a.sog.poly) {   // the polynomials' degree: 24, 26 or 28
        if (a.sog.poly <= 24) hipLaunchKernelGGL((k_near<false, ENERGY, -24>), grid, block, lds, st, a);
        else if (a.sog.poly <= 26) hipLaunchKernelGGL((k_near<false, ENERGY, -26>), grid, block, lds, st, a);
        else hipLaunchKernelGGL((k_near<false, ENERGY, kPolyNG>), grid, block, lds, st, a);
        return;
    }
    switch (a.sog.n) {
#define RBSOG_NEAR_NG(n) \
    case n: hipLaunchKernelGGL((k_near<MIXED, ENERGY, n>), grid, block, lds, st, a); return;
        RBSOG_NEAR_NG(1)
        RBSOG_NEAR_NG(2)
        RBSOG_NEAR_NG(3)
        RBSOG_NEAR_NG(4)
        RBSOG_NEAR_NG(5)
        RBSOG_NEAR_NG(6)
        RBSOG_NEAR_NG(7)
        RBSOG_NEAR_NG(8)
#undef RBSOG_NEAR_NG
    default: hipLaunchKernelGGL((k_near<MIXED, ENERGY, 0>), grid, block, lds, st, a); return;
    }
}

hipError_t launch_nlist_batch(const NearArgs *tab, const EnsItem *items, int n, hipStream_t st)
{
    if (!tab || !items || n < 1) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_nlist_batch, dim3(n), dim3(kListThreads), 0, st, tab, items);
    return hipGetLastError();
}

hipError_t launch_near_batch(const NearArgs *tab, const RhoArgs *rho, const EnsItem *items, int n, NearKind kind,
                             size_t lds, hipStream_t st)
{
    if (!tab || !rho || !items || n < 1 || lds > 65536) return hipErrorInvalidValue;
    const dim3 grid(n), block(kNearThreads);
    if (kind == NearKind::kMixed) hipLaunchKernelGGL(k_near_batch<NearKind::kMixed>, grid, block, lds, st, tab, rho, items);
    else if (kind == NearKind::kPoly)
        hipLaunchKernelGGL(k_near_batch<NearKind::kPoly>, grid, block, lds, st, tab, rho, items);
    else hipLaunchKernelGGL(k_near_batch<NearKind::kExp>, grid, block, lds, st, tab, rho, items);
    return hipGetLastError();
}

hipError_t launch_near(const NearArgs &a, hipStream_t st)
{
    if (!near_args_ok(a) || a.sog.n < 1 || a.sog.n > kMaxGauss) return hipErrorInvalidValue;
    dim3 grid(near_blocks(a.N) + a.nrho);
    if (a.mixed) {
        if (a.energy) launch_near_ng<true, true>(a, grid, st);
        else launch_near_ng<true, false>(a, grid, st);
    } else {
        if (a.energy) launch_near_ng<false, true>(a, grid, st);
        else launch_near_ng<false, false>(a, grid, st);
    }
    return hipGetLastError();
}

}  // namespace rbsog
