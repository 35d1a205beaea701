// The candidate windows of the fine grid's cell pairs, one per wave: shared by the
// neighbour-list build and the pair histogram.
#pragma once

#include <hip/hip_runtime.h>

#include "dev_common.h"

namespace rbsog {

__device__ inline double shift_of(int code, double L) { return (double)(code - 1) * L; }

// LDS written by some lanes of the wave is read by others after this.
__device__ inline void wave_lds_fence()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// The window of cell pair q: two x-adjacent cells of the fine grid (the last
// cell of a row of odd length alone) hold the home particles [h_beg, h_end);
// their candidates are the particles of 25 rows (dz, dy = -2..2) of the cells
// x0 - 2 .. x1 + 2, each row one contiguous range of the cell order or two
// where it wraps, 50 pieces at most.  Lane l < 50 describes piece l in the wave's
// tables.
// Returns false, uniformly over the wave, when q is past the last pair or the
// pair has no home particle.  A window holds each particle at most once: it is
// at most 6 cells wide in x and 5 in y and z, and the grid has at least 6.
// CENTRED: positions are taken relative to the pair's centre, so that a distance
// test can be written out as |c|^2 - 2 h.c + |h|^2 without losing its digits.
struct PairWindow {
    int h_beg, h_end, total;   // home particles; candidates (all uniform)
};

struct PairTables {            // one wave's window, by piece
    int32_t pref[64];          // exclusive prefix sums of the pieces' lengths
    int32_t first[64];         // particle index of candidate c of the piece, less c
    double shift[3][64];       // image shift less the centre
};

template <bool CENTRED>
__device__ inline bool pair_window(const CellGeom &g, const double cw[3], const int32_t *cell_start, int q,
                                   PairTables &w, double centre[3], PairWindow &win)
{
    const int lane = threadIdx.x & 63;
    const int nf = g.nc[0], nfy = g.nc[1], nfz = g.nc[2], half = (nf + 1) >> 1;
    if (q >= nfz * nfy * half) return false;
    const int row = q / half, ix = q - row * half;
    const int cz = row / nfy, cy = row - cz * nfy;
    const int x0 = 2 * ix, x1 = min(x0 + 1, nf - 1);
    const int cbase = (cz * nfy + cy) * nf;
    win.h_beg = __builtin_amdgcn_readfirstlane(cell_start[cbase + x0]);
    win.h_end = __builtin_amdgcn_readfirstlane(cell_start[cbase + x1 + 1]);
    if (win.h_beg >= win.h_end) return false;
    centre[0] = CENTRED ? (double)(x0 + 1) * cw[0] : 0.0;
    centre[1] = CENTRED ? ((double)cy + 0.5) * cw[1] : 0.0;
    centre[2] = CENTRED ? ((double)cz + 0.5) * cw[2] : 0.0;
    int ps = 0, plen = 0, xc = 1, yc = 1, zc = 1;
    if (lane < 2 * 25) {
        const int r = lane >> 1, k = lane & 1;
        int czw = cz + r / 5 - 2;
        if (czw < 0) { czw += nfz; zc = 0; } else if (czw >= nfz) { czw -= nfz; zc = 2; }
        int cyw = cy + r % 5 - 2;
        if (cyw < 0) { cyw += nfy; yc = 0; } else if (cyw >= nfy) { cyw -= nfy; yc = 2; }
        const int rb = (czw * nfy + cyw) * nf;
        const int xa = x0 - 2, xb = x1 + 2;   // at most 6 cells <= nf: one side wraps at most
        int lo = xa, hi = xb;
        bool has = k == 0;
        if (xa < 0) {
            has = true;
            if (k == 0) { lo = xa + nf; hi = nf - 1; xc = 0; } else { lo = 0; hi = xb; }
        } else if (xb > nf - 1) {
            has = true;
            if (k == 0) { hi = nf - 1; } else { lo = 0; hi = xb - nf; xc = 2; }
        }
        if (has) {
            ps = cell_start[rb + lo];
            plen = cell_start[rb + hi + 1] - ps;
        }
    }
    int incl = plen;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        int u = __shfl_up(incl, off);
        if (lane >= off) incl += u;
    }
    win.total = __builtin_amdgcn_readlane(incl, 63);
    w.pref[lane] = incl - plen;
    w.first[lane] = ps - (incl - plen);
    w.shift[0][lane] = shift_of(xc, g.L[0]) - centre[0];
    w.shift[1][lane] = shift_of(yc, g.L[1]) - centre[1];
    w.shift[2][lane] = shift_of(zc, g.L[2]) - centre[2];
    wave_lds_fence();
    return true;
}

// The piece of cell pair q's window that holds its home particles (see
// pair_window): the central row's first piece, or its second when the row
// wraps at the low x side.
__device__ inline int pair_window_home_piece(const CellGeom &g, int q)
{
    const int half = (g.nc[0] + 1) >> 1;
    const int ix = q - (q / half) * half;
    return 2 * ix - 2 < 0 ? 25 : 24;
}

// The piece of candidate c (< the window's total): the last piece whose prefix
// is <= c (an empty piece shares the prefix of the next, so it is never the
// one found), by binary search over the 64 prefixes.
__device__ inline int window_piece(const int32_t *ppref, int c)
{
    int lo = 0, n = 64;
    while (n > 0) {
        int h2 = n >> 1;
        if (ppref[lo + h2] <= c) { lo += h2 + 1; n -= h2 + 1; }
        else n = h2;
    }
    return lo - 1;
}

// Windows of up to kPieceTab candidates get a table of each candidate's piece (one
// byte each, in LDS), written once per window: a lookup per candidate in place of
// a binary search per chunk of candidates, which the few home particles of a
// cell pair (~8 at the N = 1e6 plasma) would otherwise share.  Returns whether
// the table holds them (uniform).
constexpr int kPieceTab = 2048;

__device__ inline bool window_pieces(const PairTables &w, int total, uint8_t *pidx)
{
    if (total > kPieceTab) return false;
    const int lane = threadIdx.x & 63;   // lane l writes its piece's index over the piece's candidates
    const int b0 = w.pref[lane], b1 = lane < 63 ? w.pref[lane + 1] : total;
    for (int t = b0; t < b1; ++t) pidx[t] = (uint8_t)lane;
    wave_lds_fence();
    return true;
}

}  // namespace rbsog
