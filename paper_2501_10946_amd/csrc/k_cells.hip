// gfx950 kernels of librbsog: the cell list (a counting sort with a stable
// rank), the first velocity-Verlet half step, and the moves between the
// caller's particle order and cell order.
//
// Data layout in HBM: the caller's particle arrays are FP64 SoA in the
// caller's order; the library keeps the state it steps in cell order (xs[N]
// = (x, y, z, q) as double4, 32-byte rows, velocities, forces and masses as
// SoA), with order[p] the caller index of cell position p.  Every kernel of a
// step streams these arrays contiguously; the caller's arrays are read once
// when a call starts and written once when it ends.  A build sorts the rows
// by (cell, caller index) and moves them into the new order.
//
// Builds can be gated: every build kernel takes a device flag and returns at
// once when it is zero, so the decision to rebuild (some particle moved more
// than half the list skin) is taken on the device with no host round-trip.
#include <hip/hip_runtime.h>


#include "dev_common.h"

namespace rbsog {

// A build kernel proceeds when it has no gate or its gate is raised.
__device__ inline bool gate_open(const int32_t *gate) { return gate == nullptr || *gate != 0; }

// ---------------------------------------------------------------------------
// cell list: ids + counts + chains, scan, stable rank + move.  Three launches: a
// gated step runs them all with the gate closed, each for its launch alone, and a
// build of up to 1e5 particles is bound by them too.  Two more (a pass of its own
// for the sums of the scan's tiles, a scatter of the members into their cells) took
// 20 steps of N = 1e5 from 1437 to 1500 us, an evaluation of N = 5003 from 55 to
// 62, a build of N = 1e6 from 71 to 82.
// ---------------------------------------------------------------------------

// Every kernel body takes its argument block and its workgroup index b within
// the system's grid; the single-system kernels pass blockIdx.x, the ensemble
// kernels the (replica, block) item of a work list.

// The particles of a wave are consecutive rows of the cell order before the
// build, so neighbouring lanes mostly share a cell.  run_length: the length of
// the run of equal ids that starts at this lane (live lanes form a prefix of the
// wave; at most kRunMax lanes), 0 where none starts.
constexpr int kRunBits = 5, kRunMax = 1 << kRunBits;
constexpr uint32_t kRunRow = (1u << (32 - kRunBits)) - 1u;   // a run: its first row, and its length - 1 above

__device__ inline int run_length(int id, bool live)
{
    const int lane = threadIdx.x & 63;
    const uint64_t lv = __builtin_amdgcn_ballot_w64(live);
    const int prev = __shfl_up(id, 1);
    const bool head = live && ((lane & (kRunMax - 1)) == 0 || prev != id);
    const uint64_t H = __builtin_amdgcn_ballot_w64(head);
    if (!head) return 0;
    const uint64_t above = H & ~((2ull << lane) - 1ull);   // (2 << 63) wraps to 0: no head above lane 63
    return (above ? __ffsll((long long)above) - 1 : 64 - __clzll((long long)lv)) - lane;
}

// A particle's row as it moves.
struct CellRow {
    double4 x;
    double m, v[3];
    int32_t order;
};

__device__ inline int cell_of(const CellGeom &g, const double4 &r)
{
    const int cx = cell_coord(r.x, g.inv_cell[0], g.nc[0]);
    const int cy = cell_coord(r.y, g.inv_cell[1], g.nc[1]);
    const int cz = cell_coord(r.z, g.inv_cell[2], g.nc[2]);
    return (cz * g.nc[1] + cy) * g.nc[0] + cx;
}

// Snapshot of row p for the rank pass and its cell id (stored).
__device__ inline int cell_id_of(const CellArgs &a, int p)
{
    const double4 r = a.xs[p];
    // snapshot of the row: the rank pass reads the old order from here while
    // it writes the new one in place
    a.xs_old[p] = r;
    a.order_old[p] = a.order[p];
    a.ms_old[p] = a.ms[p];
    if (a.vs)
        for (int d = 0; d < 3; ++d) a.vs_old[d * a.N + p] = a.vs[d * a.N + p];
    const int id = cell_of(a.g, r);
    a.cell_id[p] = id;
    return id;
}

__device__ inline void cell_ids_body(const CellArgs &a, int b)
{
    if (!gate_open(a.gate)) return;
    int p = b * kBlock + threadIdx.x;
    const bool live = p < a.N;
    int id = -1;
    if (live) id = cell_id_of(a, p);
    // a cell's count, and its rows as a chain of runs: the last one put in in
    // fill[cell], the one before each in tmp[its first row] (the first points at
    // what an earlier build left; a walk ends by the count)
    const int n = run_length(id, live);
    if (n > 0) {
        atomicAdd(&a.count[id], n);
        a.tmp[p] = (int32_t)atomicExch((uint32_t *)&a.fill[id], (uint32_t)p | ((uint32_t)(n - 1) << (32 - kRunBits)));
    }
    // up to a thread's worth of tiles first summed in the workgroup: rows in the
    // caller's order (a system's first build) reach every tile from every wave, and
    // their atomics queue on the few sums (37 us a build of 4 000 to 50 000
    // particles, 5 so; N = 1e6 in the order of an earlier build 42 and 30)
    const int tile = live ? id / kScanTile : -1;
    const int nt = run_length(tile, live);
    const int ntiles = scan_tiles(a.g.ncell);
    if (ntiles > kBlock) {   // uniform
        if (nt > 0) atomicAdd(&a.tile_sum[tile * kTilePad], nt);
        return;
    }
    __shared__ int32_t sum[kBlock];
    sum[threadIdx.x] = 0;
    __syncthreads();
    if (nt > 0) atomicAdd(&sum[tile], nt);
    __syncthreads();
    const int32_t v = sum[threadIdx.x];
    if (v > 0) atomicAdd(&a.tile_sum[threadIdx.x * kTilePad], v);
}

__device__ inline int32_t block_exclusive_scan_256(int32_t v, int32_t *sh, int32_t *total)
{
    int t = threadIdx.x;
    sh[t] = v;
    __syncthreads();
    for (int off = 1; off < kBlock; off <<= 1) {
        int32_t u = (t >= off) ? sh[t - off] : 0;
        __syncthreads();
        sh[t] += u;
        __syncthreads();
    }
    int32_t incl = sh[t];
    *total = sh[kBlock - 1];
    __syncthreads();
    return incl - v;
}

// Exclusive scan of the cell counts: each tile adds the sums of the tiles before
// it (150 at N = 1e6) and scans its own; also clears the counts, ready for the
// next build.
__device__ inline void scan_body(const CellArgs &a, int b)
{
    if (!gate_open(a.gate)) return;
    __shared__ int32_t sh[kBlock];
    int base = b * kScanTile + threadIdx.x * kScanPer;
    int32_t before = 0;
    for (int i = threadIdx.x; i < b; i += kBlock) before += a.tile_sum[i * kTilePad];
    int32_t c[kScanPer];
    int32_t s = 0;
#pragma unroll
    for (int k = 0; k < kScanPer; ++k) {
        c[k] = (base + k < a.g.ncell) ? a.count[base + k] : 0;
        s += c[k];
    }
    int32_t off, total;
    (void)block_exclusive_scan_256(before, sh, &off);
    int32_t run = block_exclusive_scan_256(s, sh, &total) + off;
#pragma unroll
    for (int k = 0; k < kScanPer; ++k) {
        if (base + k < a.g.ncell) {
            a.cell_start[base + k] = run;
            a.count[base + k] = 0;
        }
        run += c[k];
    }
    if (b == 0 && threadIdx.x == 0) a.cell_start[a.g.ncell] = a.N;
}

// Row p of the snapshot.
__device__ inline CellRow old_row(const CellArgs &a, int p)
{
    CellRow r;
    r.x = a.xs_old[p];
    r.order = a.order_old[p];
    r.m = a.ms_old[p];
    if (a.vs)
        for (int d = 0; d < 3; ++d) r.v[d] = a.vs_old[d * a.N + p];
    return r;
}

// A row to position pn of the new order; records the positions of the build.
__device__ inline void place_row(const CellArgs &a, const CellRow &r, int pn)
{
    a.xs[pn] = r.x;
    a.order[pn] = r.order;
    a.ms[pn] = r.m;
    a.xb[pn] = r.x.x;
    a.xb[a.N + pn] = r.x.y;
    a.xb[2 * a.N + pn] = r.x.z;
    if (a.vs)
        for (int d = 0; d < 3; ++d) a.vs[d * a.N + pn] = r.v[d];
}

// Stable position: a particle's rank within its cell is the number of cell
// members with a smaller caller index, so the new order is that of (cell,
// caller index) whatever order the chain's runs are in and whatever the old cell
// order was.  Also clears the tile sums.
__device__ inline void rank_body(const CellArgs &a, int b)
{
    if (!gate_open(a.gate)) return;
    int p = b * kBlock + threadIdx.x;
    const int ntiles = scan_tiles(a.g.ncell), threads = (a.N + kBlock - 1) / kBlock * kBlock;
    for (int i = p; i < ntiles; i += threads) a.tile_sum[i * kTilePad] = 0;
    if (p >= a.N) return;
    int c = a.cell_id[p];
    const int key = a.order_old[p];
    const int cb = a.cell_start[c];
    int r = 0;
    uint32_t run = (uint32_t)a.fill[c];
    for (int left = a.cell_start[c + 1] - cb;;) {
        const int q = (int)(run & kRunRow), n = (int)(run >> (32 - kRunBits)) + 1;
        left -= n;
        if (left > 0) run = (uint32_t)a.tmp[q];   // on its way while this run is compared
        for (int k = 0; k < n; ++k) r += (a.order_old[q + k] < key);
        if (left <= 0) break;
    }
    place_row(a, old_row(a, p), cb + r);
}

RBSOG_KERNELS(cell_ids, CellArgs, kBlock)
RBSOG_KERNELS(scan, CellArgs, kBlock)
RBSOG_KERNELS(rank, CellArgs, kBlock)

// ---------------------------------------------------------------------------
// the whole build of a small system in one workgroup: counts, their scan, the
// members of each cell and the ranks in LDS; the result is that of the passes
// above (the same stable order).  A small system's step is a chain of short
// launches that the host enqueues no faster than the GPU runs them (3.4 us
// each): with its gate closed this is one of them instead of three (N = 1000: a
// step 24 us, 32 by the passes).  A build itself is bound by what one compute unit moves:
// up to four rows per thread stay in registers (N <= 4096); more go through the
// snapshot, as in the passes, and take longer than those while the gate is open.
// ---------------------------------------------------------------------------

constexpr int kSmallThreads = 1024;
static_assert(kSmallBuildN == 4 * kSmallThreads && kSmallBuildRareN == 16 * kSmallThreads, "rows per thread");

// How many of v[from .. to) are less than key, four to a read where v is aligned: a
// thread reads all of its cell, and all of a clump's threads read all of the clump.
__device__ inline int below(const int32_t *v, int from, int to, int key)
{
    int r = 0, m = from;
    for (; m < to && (m & 3); ++m) r += v[m] < key;
    for (; m + 3 < to; m += 4) {
        const int4 u = *(const int4 *)(v + m);
        r += (u.x < key) + (u.y < key) + (u.z < key) + (u.w < key);
    }
    for (; m < to; ++m) r += v[m] < key;
    return r;
}

template <int ROWS, bool HOLD>
__global__ __launch_bounds__(kSmallThreads) void k_build_small(CellArgs a)
{
    if (!gate_open(a.gate)) return;
    constexpr int kMax = ROWS * kSmallThreads;
    __shared__ int32_t start[kSmallBuildCells];   // counts, then the cells' first positions
    __shared__ __align__(16) int32_t member[kMax];   // caller indices by cell, unordered
    __shared__ int32_t wsum[kSmallThreads / 64];
    const int t = threadIdx.x, lane = t & 63, wv = t >> 6;
    for (int c = t; c < a.g.ncell; c += kSmallThreads) start[c] = 0;
    __syncthreads();
    int id[ROWS], slot[ROWS];
    CellRow row[HOLD ? ROWS : 1];
#pragma unroll
    for (int k = 0; k < ROWS; ++k) {
        const int p = k * kSmallThreads + t;
        if (p < a.N) {
            if constexpr (HOLD) {
                row[k].x = a.xs[p];
                row[k].order = a.order[p];
                row[k].m = a.ms[p];
                if (a.vs)
                    for (int d = 0; d < 3; ++d) row[k].v[d] = a.vs[d * a.N + p];
                id[k] = cell_of(a.g, row[k].x);
            } else {
                id[k] = cell_id_of(a, p);
            }
            slot[k] = atomicAdd(&start[id[k]], 1);
        }
    }
    __syncthreads();
    // exclusive scan: thread t takes cells [t per, (t + 1) per)
    const int per = (a.g.ncell + kSmallThreads - 1) / kSmallThreads;
    int n = 0;
    for (int k = 0; k < per; ++k)
        if (t * per + k < a.g.ncell) n += start[t * per + k];
    int incl = n;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        const int u = __shfl_up(incl, off);
        if (lane >= off) incl += u;
    }
    if (lane == 63) wsum[wv] = incl;
    __syncthreads();
    int run = incl - n;
    for (int w = 0; w < wv; ++w) run += wsum[w];
    for (int k = 0; k < per; ++k) {
        const int c = t * per + k;
        if (c < a.g.ncell) {
            const int cnt = start[c];
            start[c] = run;
            a.cell_start[c] = run;
            run += cnt;
        }
    }
    if (t == 0) a.cell_start[a.g.ncell] = a.N;
    __syncthreads();
#pragma unroll
    for (int k = 0; k < ROWS; ++k) {
        const int p = k * kSmallThreads + t;
        if (p < a.N) member[start[id[k]] + slot[k]] = HOLD ? row[HOLD ? k : 0].order : a.order_old[p];
    }
    __syncthreads();   // every row has been read: the new order may overwrite them
#pragma unroll
    for (int k = 0; k < ROWS; ++k) {
        const int p = k * kSmallThreads + t;
        if (p < a.N) {
            const int cb = start[id[k]], ce = id[k] + 1 < a.g.ncell ? start[id[k] + 1] : a.N;
            const int key = HOLD ? row[HOLD ? k : 0].order : a.order_old[p];
            const int r = below(member, cb, ce, key);
            if constexpr (HOLD) place_row(a, row[k], cb + r);
            else place_row(a, old_row(a, p), cb + r);
        }
    }
}

static bool cell_args_ok(const CellArgs &a)
{
    return a.N >= 1 && a.g.nc[0] >= 1 && a.g.nc[1] >= 1 && a.g.nc[2] >= 1 && a.xs && a.order && a.xs_old && a.order_old && (!a.vs || a.vs_old) &&
           a.ms && a.ms_old && a.xb && a.cell_id && a.count && a.cell_start && a.fill && a.tmp && a.tile_sum && a.ticket;
}

hipError_t launch_cell_build(const CellArgs &a, hipStream_t st)
{
    if (!cell_args_ok(a)) return hipErrorInvalidValue;
    if (a.g.ncell <= kSmallBuildCells && a.N <= (a.rare ? kSmallBuildRareN : kSmallBuildN)) {
        if (a.N <= kSmallBuildN) hipLaunchKernelGGL((k_build_small<4, true>), dim3(1), dim3(kSmallThreads), 0, st, a);
        else hipLaunchKernelGGL((k_build_small<16, false>), dim3(1), dim3(kSmallThreads), 0, st, a);
        return hipGetLastError();
    }
    int grid = (a.N + kBlock - 1) / kBlock;
    int nt = scan_tiles(a.g.ncell);
    hipLaunchKernelGGL(k_cell_ids, dim3(grid), dim3(kBlock), 0, st, a);
    hipLaunchKernelGGL(k_scan, dim3(nt), dim3(kBlock), 0, st, a);
    hipLaunchKernelGGL(k_rank, dim3(grid), dim3(kBlock), 0, st, a);
    return hipGetLastError();
}

hipError_t launch_cell_build_batch(const CellArgs *tab, const EnsItem *per256, int n256, const EnsItem *pertile,
                                   int ntile, hipStream_t st)
{
    if (!tab || (n256 > 0 && !per256) || (ntile > 0 && !pertile)) return hipErrorInvalidValue;
    if (n256 > 0) hipLaunchKernelGGL(k_cell_ids_batch, dim3(n256), dim3(kBlock), 0, st, tab, per256);
    if (ntile > 0) hipLaunchKernelGGL(k_scan_batch, dim3(ntile), dim3(kBlock), 0, st, tab, pertile);
    if (n256 > 0) hipLaunchKernelGGL(k_rank_batch, dim3(n256), dim3(kBlock), 0, st, tab, per256);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// first half-kick + drift + wrap in cell order; raises the rebuild gate of
// this step when a particle has moved more than half the skin since the last
// build, and clears the gate of the next step (when the caller alternates two
// gates)
// ---------------------------------------------------------------------------

// (kick_drift_body is in dev_common.h: the ensemble draws its modes beside it)
__global__ __launch_bounds__(kBlock) void k_kick_drift(KickDriftArgs a) { kick_drift_body(a, (int)blockIdx.x); }

hipError_t launch_kick_drift(const KickDriftArgs &a, hipStream_t st)
{
    if (a.N < 1 || !a.xs || !a.vs || !a.fs || !a.ms || !a.xb || !a.gate || !a.flag || (a.th.on && !a.order))
        return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_kick_drift, dim3((a.N + kBlock - 1) / kBlock), dim3(kBlock), 0, st, a);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// caller order <-> cell order
// ---------------------------------------------------------------------------

__device__ inline void state_in_body(const PermArgs &a, int b)
{
    int p = b * kBlock + threadIdx.x;
    if (p >= a.N) return;
    const int i = a.order[p];
    a.xs[p] = make_double4(a.x[i], a.x[a.N + i], a.x[2 * a.N + i], a.q[i]);
    a.ms[p] = a.m[i];
    for (int d = 0; d < 3; ++d) {
        if (a.v) a.vs[d * a.N + p] = a.v[d * a.N + i];
        if (a.f) a.fs[d * a.N + p] = a.f[d * a.N + i];
    }
}

__device__ inline void state_out_body(const PermArgs &a, int b)
{
    int p = b * kBlock + threadIdx.x;
    if (p >= a.N) return;
    const int i = a.order[p];
    const double4 r = a.xs[p];
    a.x[i] = r.x;
    a.x[a.N + i] = r.y;
    a.x[2 * a.N + i] = r.z;
    for (int d = 0; d < 3; ++d) {
        if (a.v) a.v[d * a.N + i] = a.vs[d * a.N + p];
        if (a.f) a.f[d * a.N + i] = a.fs[d * a.N + p];
    }
}

__global__ __launch_bounds__(kBlock) void k_state_in(PermArgs a) { state_in_body(a, (int)blockIdx.x); }
__global__ __launch_bounds__(kBlock) void k_state_out(PermArgs a) { state_out_body(a, (int)blockIdx.x); }

hipError_t launch_state_in(const PermArgs &a, hipStream_t st)
{
    if (a.N < 1 || !a.order || !a.x || !a.q || !a.m || !a.xs || !a.ms || (a.v && !a.vs) || (a.f && !a.fs))
        return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_state_in, dim3((a.N + kBlock - 1) / kBlock), dim3(kBlock), 0, st, a);
    return hipGetLastError();
}

hipError_t launch_state_out(const PermArgs &a, hipStream_t st)
{
    if (a.N < 1 || !a.order || !a.x || !a.xs || (a.v && !a.vs) || (a.f && !a.fs)) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_state_out, dim3((a.N + kBlock - 1) / kBlock), dim3(kBlock), 0, st, a);
    return hipGetLastError();
}

__global__ __launch_bounds__(kBlock) void k_iota(int32_t *order, int N)
{
    int p = blockIdx.x * kBlock + threadIdx.x;
    if (p < N) order[p] = p;
}

// Piece blockIdx.y.  A replica's state, tables and argument blocks are some 16
// pieces of 4 bytes to megabytes: one launch over PCIe in place of as many copies,
// each of which costs the host more (4 us) than its bytes cost the link.
__global__ __launch_bounds__(kBlock) void k_copy_segs(CopySegs a)
{
    const CopySeg s = a.s[blockIdx.y];
    const uint32_t t = blockIdx.x * kBlock + threadIdx.x, step = gridDim.x * kBlock, words = s.bytes / 4;
    uint32_t *dst = (uint32_t *)s.dst;
    if (s.kind == kCopyIota) {
        for (uint32_t i = t; i < words; i += step) dst[i] = i;
        return;
    }
    const uint32_t *src = (const uint32_t *)s.src;
    uint32_t quads = 0;
    if ((((uintptr_t)s.src | (uintptr_t)s.dst) & 15) == 0) {
        quads = words / 4;
        const uint4 zero = {0, 0, 0, 0};
        for (uint32_t i = t; i < quads; i += step)
            ((uint4 *)s.dst)[i] = s.kind == kCopyZero ? zero : ((const uint4 *)s.src)[i];
    }
    for (uint32_t i = 4 * quads + t; i < words; i += step) dst[i] = s.kind == kCopyZero ? 0u : src[i];
}

hipError_t launch_copy_segs(const CopySegs &a, hipStream_t st)
{
    if (a.n < 1 || a.n > kCopySegs) return hipErrorInvalidValue;
    uint32_t most = 0;
    for (int i = 0; i < a.n; ++i) {
        const CopySeg &s = a.s[i];
        if (!s.dst || s.bytes == 0 || (s.bytes & 3) || ((uintptr_t)s.dst & 3) ||
            (s.kind == kCopyWords && (!s.src || ((uintptr_t)s.src & 3))) || s.kind < kCopyWords || s.kind > kCopyIota)
            return hipErrorInvalidValue;
        most = s.bytes > most ? s.bytes : most;
    }
    const uint32_t blocks = (most + 16 * kBlock - 1) / (16 * kBlock);   // 16 bytes a lane and turn
    hipLaunchKernelGGL(k_copy_segs, dim3(blocks < 256 ? blocks : 256, a.n), dim3(kBlock), 0, st, a);
    return hipGetLastError();
}

hipError_t launch_iota(int32_t *order, int N, hipStream_t st)
{
    if (!order || N < 1) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_iota, dim3((N + kBlock - 1) / kBlock), dim3(kBlock), 0, st, order, N);
    return hipGetLastError();
}

__global__ void k_set_int(int32_t *p, int32_t v) { *p = v; }

hipError_t launch_set_int(int32_t *p, int32_t v, hipStream_t st)
{
    if (!p) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_set_int, dim3(1), dim3(1), 0, st, p, v);
    return hipGetLastError();
}

}  // namespace rbsog
