// Geometric multigrid for the 2D regularised Newton systems (section 4.2, eq. 22-25) on gfx950:
// coarse operators of eq. (24) (cross stencil -> five points on level 1, five points -> five
// points below), multicolour block SOR passes (eq. 22), restriction, injection prolongation,
// and Gaussian elimination with partial pivoting on the coarsest grid (dense, in registers).
//
// A smoothing phase of a level (all its colour passes) is one cooperative launch wherever the level's
// rows fit the registers of the chip (k_resident2d), or most of them do (k_streamed2d); launches per
// pass (k_smooth2d_pass) take its place where a cooperative launch is not possible.  Levels of
// at most 512 cells run in one workgroup (k_bottom2d).
//
// Every level keeps its per-cell arrays in colour-blocked order (Perm2D): a colour pass of the
// smoother touches only the cells of one colour, and with the colours stored apart it reads them
// contiguously instead of pulling whole cache lines of interleaved colours.  One thread per cell
// or coarse cell; the sums run in the order of the definitions, so no result depends on the
// layout.
#include <algorithm>
#include <cstring>

#include "nmg_common.h"

namespace nmg {

template <typename T>
__device__ __forceinline__ double ld2(const T *p, long long i) { return (double)p[i]; }

// a load whose data will be evicted before it is read again (STREAM): the non-temporal hint
// keeps it out of the memory-side cache
template <bool STREAM, typename T>
__device__ __forceinline__ double lds2(const T *p)
{
    if (STREAM) return (double)__builtin_nontemporal_load(p);
    return (double)*p;
}

// stencil offsets: the cross of eq. (21) or the full 21 cells on the finest level, five points
// below (stencil_dx / stencil_dy)
__device__ __forceinline__ void stencil_off(int nb, int b, int &di, int &dj)
{
    di = stencil_dx(nb, b);
    dj = stencil_dy(nb, b);
}

__device__ constexpr int find_off(int nb, int di, int dj)
{
    for (int b = 0; b < nb; b++)
        if (stencil_dx(nb, b) == di && stencil_dy(nb, b) == dj) return b;
    return -1;
}

__device__ __forceinline__ void inv3d(const double A[9], double B[9])
{
    const double c00 = A[4] * A[8] - A[5] * A[7];
    const double c01 = A[5] * A[6] - A[3] * A[8];
    const double c02 = A[3] * A[7] - A[4] * A[6];
    const double det = A[0] * c00 + A[1] * c01 + A[2] * c02;
    B[0] = c00 / det;
    B[1] = (A[2] * A[7] - A[1] * A[8]) / det;
    B[2] = (A[1] * A[5] - A[2] * A[4]) / det;
    B[3] = c01 / det;
    B[4] = (A[0] * A[8] - A[2] * A[6]) / det;
    B[5] = (A[2] * A[3] - A[0] * A[5]) / det;
    B[6] = c02 / det;
    B[7] = (A[1] * A[6] - A[0] * A[7]) / det;
    B[8] = (A[0] * A[4] - A[1] * A[3]) / det;
}

// eq. (24), operator part, one thread per coarse cell and five-point offset BC: the sum of the fine
// blocks of the 2x2 children rows against the 2x2 children of the neighbour; for the centre also D^{-1}.
// The block of every pair of children is known at compile time, so a thread's loads (at most 16
// blocks of nine) issue together; an offset per thread, a fifth of the row each, keeps the small
// levels' few cells from being one long chain (37 -> 6.5 us for a 32 x 16 coarse level).
template <typename T, int NB, int BC>
__device__ __forceinline__ void coarsen_block(T *mg, const Level2D &Lf, const Level2D &Lc, int I, int Jq)
{
    constexpr int dP = stencil_dx(5, BC), dQ = stencil_dy(5, BC);
    const long long nf = Lf.P.M, nc = Lc.P.M;
    const long long cc = perm2d(Lc.P, I, Jq);
    const int P = I + dP, Q = Jq + dQ;
    double blk[9];
#pragma unroll
    for (int e = 0; e < 9; e++) blk[e] = 0.0;
    if (P >= 0 && P < Lc.nx && Q >= 0 && Q < Lc.ny) {
#pragma unroll
        for (int f = 0; f < 4; f++) {
            const long long fc = perm2d_rows(Lf.P, 2 * I + (f & 1), 2 * Jq + (f >> 1));
#pragma unroll
            for (int g = 0; g < 4; g++) {
                const int b = find_off(NB, 2 * dP + (g & 1) - (f & 1), 2 * dQ + (g >> 1) - (f >> 1));
                if (b < 0) continue;
#pragma unroll
                for (int e = 0; e < 9; e++) blk[e] = blk[e] + ld2(mg + Lf.J, (b * 9 + e) * nf + fc);
            }
        }
    }
#pragma unroll
    for (int e = 0; e < 9; e++) mg[Lc.J + (BC * 9 + e) * nc + cc] = (T)blk[e];
    if (BC == 0) {
        double B[9];
        inv3d(blk, B);
#pragma unroll
        for (int e = 0; e < 9; e++) mg[Lc.Dinv + e * nc + cc] = (T)B[e];
    }
}

template <typename T, int NB>
__global__ void __launch_bounds__(64) k_coarsen2d(T *mg, Level2D Lf, Level2D Lc)
{
    const int I = blockIdx.x * 64 + threadIdx.x, Jq = blockIdx.y;
    if (I >= Lc.nx) return;
    switch (blockIdx.z) {
    case 0: coarsen_block<T, NB, 0>(mg, Lf, Lc, I, Jq); break;
    case 1: coarsen_block<T, NB, 1>(mg, Lf, Lc, I, Jq); break;
    case 2: coarsen_block<T, NB, 2>(mg, Lf, Lc, I, Jq); break;
    case 3: coarsen_block<T, NB, 3>(mg, Lf, Lc, I, Jq); break;
    default: coarsen_block<T, NB, 4>(mg, Lf, Lc, I, Jq); break;
    }
}

// A launch per colour pass over a level whose rows lie in tiles: a wavefront takes 64 rows of the tile
// (column blockIdx.z, row blockIdx.x of tiles) and colour, the blockIdx.y-th 64 from a multiple of 16 on
// (from anywhere else a load takes twice the accesses of the first-level cache).  dU is in the order
// without tiles, and its cache lines cross from a tile to the next in its row: with blockIdx.x along the
// column, the tiles of a row mostly fall to one XCD, whose L2 then writes whole lines (1024 x 512, a pass:
// FP32 15.0 us with the row's tiles on all XCDs, 12.7 so; FP64 17.1 to 26.8, 16.8 to 25.7).
// (i, j), row: the cell of lane p; false: the tile has none there.
constexpr int kTileRows = 64, kRowAlign = 16;

__device__ __forceinline__ bool tiled_cell(const Level2D &L, int colour, int p, int &i, int &j, int &row)
{
    const int i0 = blockIdx.z * L.P.tw(), j0 = blockIdx.x * L.P.th();
    const int w = L.nx - i0 < L.P.tw() ? L.nx - i0 : L.P.tw(), h = L.ny - j0 < L.P.th() ? L.ny - j0 : L.P.th();
    const int start = (int)tile3_start(L.P, colour, i0, j0, h);
    row = (start & -kRowAlign) + blockIdx.y * kTileRows + p;
    const int e = row - start;
    if (e < 0 || e >= tile3_count(colour, i0, j0, w, h)) return false;
    int il, jr;
    tile3_cell(colour, i0, j0, w, e, il, jr);
    i = i0 + il;
    j = j0 + jr;
    return true;
}

// `reps` consecutive passes of eq. (22) over the cells of one colour on one level with the
// NB-block stencil (C = 3 colours (i + j) mod 3 for the nine-block cross, 2 for five points, 9
// colours (i mod 3) + 3 (j mod 3) for the full 21 cells), thread p taking slot p of that colour's
// block (row p / W, k-th cell of the colour in the row; tiled_cell where the rows lie in tiles).  Passes
// of one colour in a row see the same neighbour values, so the off-diagonal sum and D^{-1} r are
// formed once and the relaxation is applied `reps` times, each result rounded to the storage
// type as if it had been stored between the passes.  The stencil is unrolled so that every load
// of the cell's row is issued up front; neighbours outside the grid read the cell's own slot and
// are left out of the sum.
// TILED: the level's rows lie in tiles (NB = 9)
template <typename T, int NB, bool STREAM = false>
__device__ __forceinline__ void smooth_slot21(T *mg, const Level2D &L, int colour, double omega, int reps, long long p);

template <typename T, int NB, bool STREAM = false, bool TILED = false>
__device__ __forceinline__ void smooth_slot(T *mg, const Level2D &L, int colour, double omega, int reps, long long p)
{
    if constexpr (NB == 21) {
        smooth_slot21<T, NB, STREAM>(mg, L, colour, omega, reps, p);
        return;
    } else {
    constexpr int C = NB == 9 ? 3 : 2;
    const int W = L.P.W;
    int i, j;
    long long cc, rr;                            // dU of the cell, its row
    if constexpr (TILED) {
        int row;
        if (!tiled_cell(L, colour, (int)p, i, j, row)) return;
        rr = row;
        cc = perm2d_of<C>(L.P, i, j);
    } else {
        if (p >= (long long)L.P.ny * W) return;
        j = (int)(p / W);
        i = ((colour - j) % C + C) % C + C * (int)(p - (long long)j * W);
        if (i >= L.nx) return;
        cc = rr = (long long)colour * L.P.ny * W + p;
    }
    const long long n = L.P.M;
    const T *Jr = mg + L.J + rr;
    const T *Ur = mg + L.dU;
    double x[NB][3];
    bool ok[NB];
#pragma unroll
    for (int b = 1; b < NB; b++) {
        int di, dj;
        stencil_off(NB, b, di, dj);
        const int pi = i + di, pj = j + dj;
        ok[b] = pi >= 0 && pi < L.nx && pj >= 0 && pj < L.ny;
        const int c2 = (colour + di + dj + 2 * C) % C;           // the neighbour's colour, the same in every lane
        const long long q = ok[b] ? (long long)c2 * L.ny * W + (long long)pj * W + pi / C : cc;
#pragma unroll
        for (int c = 0; c < 3; c++) x[b][c] = (double)Ur[c * n + q];
    }
    double a[NB][3];
#pragma unroll
    for (int b = 1; b < NB; b++)
#pragma unroll
        for (int c = 0; c < 3; c++)
            a[b][c] = lds2<STREAM>(Jr + (b * 9 + c * 3 + 0) * n) * x[b][0] + lds2<STREAM>(Jr + (b * 9 + c * 3 + 1) * n) * x[b][1] +
                      lds2<STREAM>(Jr + (b * 9 + c * 3 + 2) * n) * x[b][2];
    double r[3];
#pragma unroll
    for (int c = 0; c < 3; c++) {
        r[c] = ld2(mg + L.rhs, c * n + rr);
#pragma unroll
        for (int b = 1; b < NB; b++)
            if (ok[b]) r[c] = r[c] + a[b][c];
    }
    double t[3];
#pragma unroll
    for (int c = 0; c < 3; c++)
        t[c] = lds2<STREAM>(mg + L.Dinv + (c * 3 + 0) * n + rr) * r[0] + lds2<STREAM>(mg + L.Dinv + (c * 3 + 1) * n + rr) * r[1] +
               lds2<STREAM>(mg + L.Dinv + (c * 3 + 2) * n + rr) * r[2];
#pragma unroll
    for (int c = 0; c < 3; c++) {
        T d = mg[L.dU + c * n + cc];
        for (int q = 0; q < reps; q++) d = (T)((1.0 - omega) * (double)d - omega * t[c]);
        mg[L.dU + c * n + cc] = d;
    }
    }
}

// The same pass on the full 21-cell stencil with nine colours: thread p is cell
// (3 (p mod W) + colour mod 3, 3 (p / W) + colour / 3).  The off-diagonal sum runs block by block
// in stencil order (the order of eq. 22's sum as the oracle forms it), each block's three
// products added before the block joins the sum; the blocks' loads are independent of the sum,
// so they issue ahead of it.
template <typename T, int NB, bool STREAM>
__device__ __forceinline__ void smooth_slot21(T *mg, const Level2D &L, int colour, double omega, int reps, long long p)
{
    const int W = L.P.W;
    if (p >= (long long)L.P.ny * W) return;
    const int jr = (int)(p / W), k = (int)(p - (long long)jr * W);
    const int i = 3 * k + colour % 3, j = 3 * jr + colour / 3;
    if (i >= L.nx || j >= L.ny) return;
    const long long n = L.P.M, cc = (long long)colour * L.P.ny * W + p;
    const T *Jr = mg + L.J + cc;
    const T *Ur = mg + L.dU;
    double r[3];
#pragma unroll
    for (int c = 0; c < 3; c++) r[c] = ld2(mg + L.rhs, c * n + cc);
#pragma unroll
    for (int b = 1; b < 21; b++) {
        int di, dj;
        stencil_off(21, b, di, dj);
        const int pi = i + di, pj = j + dj;
        const bool ok = pi >= 0 && pi < L.nx && pj >= 0 && pj < L.ny;
        const long long q = ok ? perm2d_of<9>(L.P, pi, pj) : cc;
        const double x0 = (double)Ur[q], x1 = (double)Ur[n + q], x2 = (double)Ur[2 * n + q];
#pragma unroll
        for (int c = 0; c < 3; c++) {
            const double a = lds2<STREAM>(Jr + (b * 9 + c * 3 + 0) * n) * x0 + lds2<STREAM>(Jr + (b * 9 + c * 3 + 1) * n) * x1 +
                             lds2<STREAM>(Jr + (b * 9 + c * 3 + 2) * n) * x2;
            if (ok) r[c] = r[c] + a;
        }
    }
    double t[3];
#pragma unroll
    for (int c = 0; c < 3; c++)
        t[c] = lds2<STREAM>(mg + L.Dinv + (c * 3 + 0) * n + cc) * r[0] + lds2<STREAM>(mg + L.Dinv + (c * 3 + 1) * n + cc) * r[1] +
               lds2<STREAM>(mg + L.Dinv + (c * 3 + 2) * n + cc) * r[2];
#pragma unroll
    for (int c = 0; c < 3; c++) {
        T d = mg[L.dU + c * n + cc];
        for (int q = 0; q < reps; q++) d = (T)((1.0 - omega) * (double)d - omega * t[c]);
        mg[L.dU + c * n + cc] = d;
    }
}

// (FP32 cross: at most 128 registers, for four wavefronts a SIMD; with rows in tiles 132 without the bound)
template <typename T, int NB, bool STREAM, bool TILED = false>
__global__ void __launch_bounds__(256, sizeof(T) == 4 && NB == 9 ? 4 : 1) k_smooth2d_pass(T *mg, Level2D L, int colour, double omega, int reps)
{
    const long long first = TILED ? 0 : blockIdx.x * (long long)blockDim.x;
    smooth_slot<T, NB, STREAM, TILED>(mg, L, colour, omega, reps, first + threadIdx.x);
}

// The same passes with each cell's three rows of eq. (22) on three lanes: wavefront c of a
// 192-thread workgroup forms row c (the off-diagonal sum in stencil order, as the per-cell form
// does) for 64 consecutive slots of the colour, so every wavefront reads one row of the blocks
// at consecutive addresses; the three sums meet in LDS, and lane c applies row c of D^{-1} and
// relaxes component c.  The same operations in the same order as smooth_slot, so the results
// are identical; three times the threads of the per-cell form, and a third of its loads per
// thread, keep more of a colour's cells in flight.
constexpr int kSplitCells = 64;
static_assert(kSplitCells == kTileRows, "one chunk of a tile's rows a workgroup");

template <typename T, int NB, bool STREAM, bool TILED = false>
__global__ void __launch_bounds__(3 * kSplitCells) k_smooth2d_split(T *mg, Level2D L, int colour, double omega, int reps)
{
    __shared__ double sr[3][kSplitCells];
    constexpr int C = NB == 9 ? 3 : (NB == 21 ? 9 : 2);
    const int c = threadIdx.x / kSplitCells, lane = threadIdx.x % kSplitCells;
    const long long p = blockIdx.x * (long long)kSplitCells + lane;
    const int W = L.P.W;
    bool valid = TILED || p < (long long)L.P.ny * W;
    int i = 0, j = 0;
    long long cc = (long long)colour * L.P.ny * W + p, rr = cc;  // dU of the cell, its row
    if (valid) {
        if constexpr (TILED) {
            int row;
            valid = tiled_cell(L, colour, lane, i, j, row);
            if (valid) { rr = row; cc = perm2d_of<C>(L.P, i, j); }
        } else {
            const int jr = (int)(p / W), k = (int)(p - (long long)jr * W);
            if (C == 9) { i = 3 * k + colour % 3; j = 3 * jr + colour / 3; }
            else { j = jr; i = ((colour - j) % C + C) % C + C * k; }
            valid = i < L.nx && j < L.ny;
        }
    }
    const long long n = L.P.M;
    double r = 0.0;
    if (valid) {
        const T *Jr = mg + L.J + rr;
        const T *Ur = mg + L.dU;
        r = ld2(mg + L.rhs, c * n + rr);
#pragma unroll
        for (int b = 1; b < NB; b++) {
            int di, dj;
            stencil_off(NB, b, di, dj);
            const int pi = i + di, pj = j + dj;
            const bool ok = pi >= 0 && pi < L.nx && pj >= 0 && pj < L.ny;
            const long long q = ok ? perm2d_of<C>(L.P, pi, pj) : cc;
            const double a = lds2<STREAM>(Jr + (b * 9 + c * 3 + 0) * n) * (double)Ur[q] +
                             lds2<STREAM>(Jr + (b * 9 + c * 3 + 1) * n) * (double)Ur[n + q] +
                             lds2<STREAM>(Jr + (b * 9 + c * 3 + 2) * n) * (double)Ur[2 * n + q];
            if (ok) r = r + a;
        }
    }
    sr[c][lane] = r;
    __syncthreads();
    if (!valid) return;
    const double t = lds2<STREAM>(mg + L.Dinv + (c * 3 + 0) * n + rr) * sr[0][lane] +
                     lds2<STREAM>(mg + L.Dinv + (c * 3 + 1) * n + rr) * sr[1][lane] +
                     lds2<STREAM>(mg + L.Dinv + (c * 3 + 2) * n + rr) * sr[2][lane];
    T d = mg[L.dU + c * n + cc];
    for (int q = 0; q < reps; q++) d = (T)((1.0 - omega) * (double)d - omega * t);
    mg[L.dU + c * n + cc] = d;
}

// ---- the four directional sweeps D1-D4 of section 4.2 (eq. 22 in a lexicographic order) ------

// eq. (22) for cell (i, j) in place, by a team of TEAM lanes (TEAM >= NB - 1, a power of two
// within one wavefront): lane m loads off-diagonal block b = m + 1 and the current dU of that
// neighbour and forms its product, all lanes at once (the loads of a hyperplane are one round
// trip, not NB - 1 of them); lane 0 of the team then adds the products to rhs in stencil order,
// skipping neighbours outside the grid, exactly the sequential sum, and writes
// dU <- (1 - omega) dU - omega D^{-1} r
template <typename T, int NB, int TEAM>
__device__ __forceinline__ void relax_cell_team(T *mg, const Level2D &L, int i, int j, double omega, int m)
{
    const long long n = L.P.M, cc = perm2d_of<colours2d(NB)>(L.P, i, j);
    const int b = m + 1;
    double a0 = 0.0, a1 = 0.0, a2 = 0.0;
    if (b < NB) {
        int di, dj;
        stencil_off(NB, b, di, dj);
        const int pi = i + di, pj = j + dj;
        if (pi >= 0 && pi < L.nx && pj >= 0 && pj < L.ny) {
            const T *Jr = mg + L.J + cc;
            const T *Ur = mg + L.dU;
            const long long q = perm2d_of<colours2d(NB)>(L.P, pi, pj);
            const double x0 = (double)Ur[q], x1 = (double)Ur[n + q], x2 = (double)Ur[2 * n + q];
            a0 = (double)Jr[(b * 9 + 0) * n] * x0 + (double)Jr[(b * 9 + 1) * n] * x1 + (double)Jr[(b * 9 + 2) * n] * x2;
            a1 = (double)Jr[(b * 9 + 3) * n] * x0 + (double)Jr[(b * 9 + 4) * n] * x1 + (double)Jr[(b * 9 + 5) * n] * x2;
            a2 = (double)Jr[(b * 9 + 6) * n] * x0 + (double)Jr[(b * 9 + 7) * n] * x1 + (double)Jr[(b * 9 + 8) * n] * x2;
        }
    }
    double r0 = 0.0, r1 = 0.0, r2 = 0.0, Di[9], d0 = 0.0, d1 = 0.0, d2 = 0.0;
    if (m == 0) {
        r0 = ld2(mg + L.rhs, cc);
        r1 = ld2(mg + L.rhs, n + cc);
        r2 = ld2(mg + L.rhs, 2 * n + cc);
#pragma unroll
        for (int e = 0; e < 9; e++) Di[e] = ld2(mg + L.Dinv, e * n + cc);
        d0 = ld2(mg + L.dU, cc);
        d1 = ld2(mg + L.dU, n + cc);
        d2 = ld2(mg + L.dU, 2 * n + cc);
    }
#pragma unroll
    for (int bb = 1; bb < NB; bb++) {
        const double v0 = __shfl(a0, bb - 1, TEAM), v1 = __shfl(a1, bb - 1, TEAM), v2 = __shfl(a2, bb - 1, TEAM);
        int di, dj;
        stencil_off(NB, bb, di, dj);
        const int pi = i + di, pj = j + dj;
        if (pi >= 0 && pi < L.nx && pj >= 0 && pj < L.ny) {
            r0 = r0 + v0;
            r1 = r1 + v1;
            r2 = r2 + v2;
        }
    }
    if (m != 0) return;
    const double t0 = Di[0] * r0 + Di[1] * r1 + Di[2] * r2;
    const double t1 = Di[3] * r0 + Di[4] * r1 + Di[5] * r2;
    const double t2 = Di[6] * r0 + Di[7] * r1 + Di[8] * r2;
    mg[L.dU + cc] = (T)((1.0 - omega) * d0 - omega * t0);
    mg[L.dU + n + cc] = (T)((1.0 - omega) * d1 - omega * t1);
    mg[L.dU + 2 * n + cc] = (T)((1.0 - omega) * d2 - omega * t2);
}

// nu smoothing iterations of the sweeps D1 (x ascending, y ascending inside), D2 (x descending),
// D3 (both descending), D4 (y descending) on one level, by one workgroup.  In the coordinates
// (i', j') of a sweep (i' the outer index) a cell needs the new values of the coupled cells with
// A i' + j' smaller and the old ones of those with it larger (A = 1 for the cross and five-point
// stencils, 3 for the full 21 cells, whose couplings reach (1, -2)); the cells of one hyperplane
// A i' + j' = h are not coupled, so the hyperplanes run in order, each in parallel (a team of
// lanes per cell): the same result as the sequential sweep, bit for bit.
template <typename T, int NB>
__device__ void sweeps_level(T *mg, const Level2D &L, int nu, double omega)
{
    constexpr int A = NB == 21 ? 3 : 1;
    constexpr int TEAM = NB == 21 ? 32 : (NB == 9 ? 8 : 4);
    static_assert(TEAM >= NB - 1 && 64 % TEAM == 0, "a team per cell inside one wavefront");
    const int nx = L.nx, ny = L.ny, H = A * (nx - 1) + ny;
    const int team = (int)threadIdx.x / TEAM, m = (int)threadIdx.x % TEAM, teams = (int)blockDim.x / TEAM;
    for (int it = 0; it < nu; it++)
        for (int d = 0; d < 4; d++) {
            const bool fi = d == 1 || d == 2, fj = d >= 2;
            for (int h = 0; h < H; h++) {
                const int lo = h - (ny - 1) > 0 ? (h - (ny - 1) + A - 1) / A : 0;
                const int hi = nx - 1 < h / A ? nx - 1 : h / A;
                for (int k = lo + team; k <= hi; k += teams) {
                    const int jp = h - A * k;
                    relax_cell_team<T, NB, TEAM>(mg, L, fi ? nx - 1 - k : k, fj ? ny - 1 - jp : jp, omega, m);
                }
                __syncthreads();
            }
        }
}

template <typename T, int NB>
__global__ void __launch_bounds__(1024) k_sweeps2d(T *mg, Level2D L, int nu, double omega)
{
    sweeps_level<T, NB>(mg, L, nu, omega);
}

// eq. (24), right-hand side of coarse cell (I, Jq); also clears its dU.
// rhs + J dU of fine cell (fi, fj), the summand of eq. (24)'s restriction
template <typename T>
__device__ __forceinline__ void restrict_child(const T *mg, const Level2D &Lf, int fi, int fj, double a[3])
{
    const long long nf = Lf.P.M;
    const long long fc = perm2d_rows(Lf.P, fi, fj);
#pragma unroll
    for (int c = 0; c < 3; c++) a[c] = ld2(mg + Lf.rhs, c * nf + fc);
    for (int b = 0; b < Lf.nb; b++) {
        int di, dj;
        stencil_off(Lf.nb, b, di, dj);
        const int pi = fi + di, pj = fj + dj;
        if (pi < 0 || pi >= Lf.nx || pj < 0 || pj >= Lf.ny) continue;
        const long long q = perm2d(Lf.P, pi, pj);
        const double x0 = ld2(mg + Lf.dU, q), x1 = ld2(mg + Lf.dU, nf + q), x2 = ld2(mg + Lf.dU, 2 * nf + q);
#pragma unroll
        for (int c = 0; c < 3; c++)
            a[c] = a[c] + (ld2(mg + Lf.J, (b * 9 + c * 3 + 0) * nf + fc) * x0 +
                           ld2(mg + Lf.J, (b * 9 + c * 3 + 1) * nf + fc) * x1 +
                           ld2(mg + Lf.J, (b * 9 + c * 3 + 2) * nf + fc) * x2);
    }
}

// coarse rhs = the four children's summands added in the order (2I, 2J), (2I+1, 2J), (2I, 2J+1),
// (2I+1, 2J+1); coarse dU = 0
template <typename T>
__device__ __forceinline__ void restrict_store(T *mg, const Level2D &Lc, int I, int Jq, const double a00[3],
                                               const double a10[3], const double a01[3], const double a11[3])
{
    const long long nc = Lc.P.M, cc = perm2d(Lc.P, I, Jq);
#pragma unroll
    for (int c = 0; c < 3; c++) {
        double sum = 0.0;
        sum = sum + a00[c];
        sum = sum + a10[c];
        sum = sum + a01[c];
        sum = sum + a11[c];
        mg[Lc.rhs + c * nc + cc] = (T)sum;
        mg[Lc.dU + c * nc + cc] = (T)0.0;
    }
}

template <typename T>
__device__ __forceinline__ void restrict_cell(T *mg, const Level2D &Lf, const Level2D &Lc, int I, int Jq)
{
    double a00[3], a10[3], a01[3], a11[3];
    restrict_child(mg, Lf, 2 * I, 2 * Jq, a00);
    restrict_child(mg, Lf, 2 * I + 1, 2 * Jq, a10);
    restrict_child(mg, Lf, 2 * I, 2 * Jq + 1, a01);
    restrict_child(mg, Lf, 2 * I + 1, 2 * Jq + 1, a11);
    restrict_store(mg, Lc, I, Jq, a00, a10, a01, a11);
}

// One workgroup per strip of two fine rows and kRX fine columns: a thread per fine cell forms its
// summand (consecutive lanes read consecutive slots of the colour-blocked arrays), then a thread
// per coarse cell adds its four children from LDS.
constexpr int kRX = 128;

template <typename T>
__global__ void __launch_bounds__(2 * kRX) k_restrict2d(T *mg, Level2D Lf, Level2D Lc)
{
    __shared__ double sa[3][2][kRX];
    const int t = threadIdx.x, r = t / kRX, x = t % kRX;
    const int fi = blockIdx.x * kRX + x, fj = 2 * blockIdx.y + r;
    if (fi < Lf.nx && fj < Lf.ny) {
        double a[3];
        restrict_child(mg, Lf, fi, fj, a);
#pragma unroll
        for (int c = 0; c < 3; c++) sa[c][r][x] = a[c];
    }
    __syncthreads();
    const int I = blockIdx.x * (kRX / 2) + t, Jq = blockIdx.y;
    if (t < kRX / 2 && I < Lc.nx && Jq < Lc.ny) {
        double a00[3], a10[3], a01[3], a11[3];
#pragma unroll
        for (int c = 0; c < 3; c++) {
            a00[c] = sa[c][0][2 * t];
            a10[c] = sa[c][0][2 * t + 1];
            a01[c] = sa[c][1][2 * t];
            a11[c] = sa[c][1][2 * t + 1];
        }
        restrict_store(mg, Lc, I, Jq, a00, a10, a01, a11);
    }
}

// eq. (25): dU_fine += dU_coarse(parent)
template <typename T>
__device__ __forceinline__ void prolong_cell(T *mg, const Level2D &Lf, const Level2D &Lc, int i, int j)
{
    const long long nf = Lf.P.M, nc = Lc.P.M;
    const long long fc = perm2d(Lf.P, i, j), pc = perm2d(Lc.P, i >> 1, j >> 1);
#pragma unroll
    for (int c = 0; c < 3; c++)
        mg[Lf.dU + c * nf + fc] = (T)(ld2(mg + Lf.dU, c * nf + fc) + ld2(mg + Lc.dU, c * nc + pc));
}

template <typename T>
__global__ void k_prolong2d(T *mg, Level2D Lf, Level2D Lc)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    const int j = blockIdx.y * blockDim.y + threadIdx.y;
    if (i >= Lf.nx || j >= Lf.ny) return;
    prolong_cell(mg, Lf, Lc, i, j);
}

// ---- resident smoothing of a level ----------------------------------------------------------

// One launch per smoothing phase of a level: each workgroup owns a tile of tx x ty cells, every
// thread keeps the operator rows of its cells (off-diagonal blocks, D^{-1}, right-hand side) in
// registers for all the phase's colour passes, and dU of the tile with its halo lives in LDS.
// What bounds the launched passes below is the launch itself (4-5 us each) on small levels and
// re-reading the operator 4 nu (C-1) + 1 times on large ones; here the operator is read once and
// a pass costs its arithmetic and a share of an exchange.
//
// Exchange: after every m passes a workgroup publishes its cells within the halo width of its
// edges in a mailbox and fetches its own halo from there.  A value travels as 64-bit words of 32
// payload bits under the 32-bit number of the exchange, so a word is its own arrival flag: no
// fence, no separate flag, one trip (about 1.0 us between any two workgroups of the chip, measured
// with 16 to 256 of them).  Between exchanges the workgroup also relaxes the cells of its halo that
// later passes of the group need (overlapped tiles: the compute region is the tile widened by
// R (m-1) cells, R the reach of the stencil; dU is held R m cells wide), so the exchanges are
// fewer and each result is formed from the same values by the same operations as in the
// launched passes, bit for bit.
//
// Two parities of the mailbox suffice: a workgroup writes exchange e + 2 only after it has fetched
// e + 1 from every workgroup whose cells its halo holds, which are those whose halos hold its cells, and
// each of them published e + 1 after it had fetched e.  The exchanges also order the phase's memory: a
// workgroup loads dU of its tile and halo (and the parents' dU) at the start and writes its tile's dU
// (and clears its parents') in place at the end, so between the two it has to have heard from every
// neighbour, which each has loaded before it publishes.  Hence a phase has at least one exchange: one
// that ends without (no restriction) exchanges before its last pass at the latest (phase2d), and one
// without passes is not run here.  A halo leaves out its corners, which m
// passes of a cross stencil do not reach.  With m = 1 only the pass's colour is exchanged (tiles are
// at least two cells wide, so every shared edge holds every colour), with m >= 2 every cell.
//
// The launch is cooperative, so all workgroups are resident and every wait ends; each wait is
// bounded all the same (kWaitTicks of the 100 MHz clock), and a workgroup whose wait ran out stops
// waiting, finishes and stores NaN.
struct Resident2DArgs {
    Level2D L, Lc;             // the level and the next coarser one
    int tx, ty, gx, m;
    int nu;                    // smoothing iterations (two phases in a row are one longer phase)
    int prolong, restr;        // eq. (25) first; eq. (24)'s right-hand side last
    unsigned tag;              // the launch's exchanges are numbered tag + 1, tag + 2, ...
    double omega;
    unsigned long long *box;   // [2][words per cell][cells]: consecutive cells' words lie together
    long long cells;
    const NewtonState *state;  // may be null: run regardless
};

constexpr long long kWaitTicks = 2000000000LL;   // 20 s

template <typename T> struct BoxWords;
template <> struct BoxWords<float> { static constexpr int n = 3; };
template <> struct BoxWords<double> { static constexpr int n = 6; };

__device__ __forceinline__ void box_put(unsigned long long *w, unsigned tag, unsigned payload)
{
    __hip_atomic_store(w, ((unsigned long long)tag << 32) | payload, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

__device__ __forceinline__ void box_store(unsigned long long *w, long long cells, unsigned tag, int c, float v)
{
    box_put(w + c * cells, tag, __float_as_uint(v));
}

__device__ __forceinline__ void box_store(unsigned long long *w, long long cells, unsigned tag, int c, double v)
{
    const unsigned long long b = (unsigned long long)__double_as_longlong(v);
    box_put(w + 2 * c * cells, tag, (unsigned)b);
    box_put(w + (2 * c + 1) * cells, tag, (unsigned)(b >> 32));
}

__device__ __forceinline__ void box_value(const unsigned long long *v, int c, float &x) { x = __uint_as_float((unsigned)v[c]); }
__device__ __forceinline__ void box_value(const unsigned long long *v, int c, double &x)
{
    x = __longlong_as_double((long long)((v[2 * c + 1] << 32) | (v[2 * c] & 0xffffffffULL)));
}

// LDS tile of dU: the cells of the tile and its halo, row by row, inside a ring of two zero cells
// (a neighbour outside the grid reads a zero of the ring).  A cell's components lie together, so that
// it is one or two LDS reads.
constexpr int kResPL = 1872;                     // cells, ring included (48 x 32 cells fit)
template <typename T> struct ResCell;
template <> struct ResCell<double> { double v[3]; };
template <> struct alignas(16) ResCell<float> { float v[4]; };
// the memory of a tile, first of its cells and then of the restriction's summands
struct alignas(16) ResLds { double v[3 * kResPL]; };
static_assert(alignof(ResLds) >= alignof(ResCell<float>) && alignof(ResLds) >= alignof(ResCell<double>) &&
                  sizeof(ResLds) >= kResPL * sizeof(ResCell<float>) && sizeof(ResLds) >= kResPL * sizeof(ResCell<double>),
              "a cell is read at its own alignment");
constexpr int kResNT = 512;
constexpr int kResHalo = 3;                      // halo cells a thread fetches at most

// a tile of w x h cells fits the plane
__host__ __device__ inline bool resident2d_fits(int w, int h) { return (w + 4) * (h + 4) <= kResPL; }

// A row held in FP32 is widened where it is used: the compiler must not widen it once before the
// passes (the FP64 copies would not fit the registers), so the value is made opaque there.
__device__ __forceinline__ void keep_narrow(float &v) { asm volatile("" : "+v"(v)); }
__device__ __forceinline__ void keep_narrow(double &) {}

// A thread has one or two cells of the five-point and cross levels; of a level with the full 21-cell
// stencil, whose rows take 192 values, it has one of a cell's three rows, the cell's rows in adjacent
// lanes (21 cells in 63 lanes of a wavefront), which hand each other their sums before D^{-1}.
constexpr int kRes21Cells = kResNT / 64 * 21;    // cells a workgroup holds then

// One smoothing phase of one level by the workgroups that share it; this one has tile (bi, bj).
// HT: the type the rows are held in; EPT: cells per thread; SOLO: one workgroup has the whole
// level (no halo, no mailbox).  dead: set when a wait ran out.
template <typename T, int NB, typename HT, int EPT, bool SOLO>
__device__ __forceinline__ void resident_level(T *mg, const Resident2DArgs &A, int bi, int bj, ResLds &lds, int &dead)
{
    constexpr int C = NB == 21 ? 9 : (NB == 9 ? 3 : 2), R = NB == 5 ? 1 : 2, NW = BoxWords<T>::n;
    constexpr int ROWS = NB == 21 ? 1 : 3;       // rows of a cell that a thread has
    static_assert(ROWS == 3 || EPT == 1, "a row a thread");
    constexpr int KB = NW == 3 ? 3 : 2;          // halo cells whose words a thread has in flight
    typedef ResCell<T> Cell;
    Cell *const sz = (Cell *)lds.v;              // dU [rows + 4][ld]; the restriction's summands last
    const Level2D &L = A.L;
    const int t = threadIdx.x, nx = L.nx, ny = L.ny;
    const int i0 = SOLO ? 0 : bi * A.tx, j0 = SOLO ? 0 : bj * A.ty;
    const int i1 = !SOLO && i0 + A.tx < nx ? i0 + A.tx : nx, j1 = !SOLO && j0 + A.ty < ny ? j0 + A.ty : ny;
    const int hc = SOLO ? 0 : R * (A.m - 1), hd = SOLO ? 0 : R * A.m;
    const int ci0 = i0 - hc > 0 ? i0 - hc : 0, ci1 = i1 + hc < nx ? i1 + hc : nx;
    const int cj0 = j0 - hc > 0 ? j0 - hc : 0, cj1 = j1 + hc < ny ? j1 + hc : ny;
    const int di0 = i0 - hd > 0 ? i0 - hd : 0, di1 = i1 + hd < nx ? i1 + hd : nx;
    const int dj0 = j0 - hd > 0 ? j0 - hd : 0, dj1 = j1 + hd < ny ? j1 + hd : ny;
    const int dw = di1 - di0, dh = dj1 - dj0, ld = dw + 4;
    Cell *const su = sz + 2 * ld + 2;
    const long long n = L.P.M;
    if (t == 0 && !SOLO) dead = 0;

    // the thread's cells: the compute region colour by colour, row by row, without gaps (C rows in a
    // row hold cw cells of every colour (i + j) mod C; the nine colours of the full stencil are the
    // pairs (i mod 3, j mod 3))
    const int cw = ci1 - ci0, ch = cj1 - cj0;
    auto first = [&](int c, int jr) { return ((c - (ci0 + cj0 + jr)) % C + C) % C; };   // column in the region
    auto first3 = [](int c, int x0) { return x0 + (c + 3 - x0 % 3) % 3; };              // first x >= x0, x mod 3 = c
    int end[C];                                  // cells of colours 0 .. c
#pragma unroll
    for (int c = 0; c < C; c++) {
        int m;
        if constexpr (NB == 21) {
            m = ((ci1 - first3(c % 3, ci0) + 2) / 3) * ((cj1 - first3(c / 3, cj0) + 2) / 3);
        } else {
            m = (ch / C) * cw;
            for (int jr = ch - ch % C; jr < ch; jr++) m += (cw - first(c, jr) + C - 1) / C;
        }
        end[c] = (c > 0 ? end[c - 1] : 0) + m;
    }
    const int lane = t & 63, row = ROWS == 1 ? lane % 3 : 0;
    HT Jb[EPT][NB][3 * ROWS], Di[EPT][3 * ROWS], rh[EPT][ROWS];
    // a cell's colour (-1: none), whether it is the tile's own and whether other tiles read it (the
    // registers are full: its place in the level is worked out from q where it is needed)
    int q[EPT], flags[EPT];
    auto colour = [&](int k) { return (flags[k] & 15) - 1; };
    auto inside = [&](int k) { return (flags[k] & 16) != 0; };
    auto edge = [&](int k) { return (flags[k] & 32) != 0; };
    auto cell_i = [&](int k) { return di0 + q[k] % ld; };
    auto cell_j = [&](int k) { return dj0 + q[k] / ld; };
#pragma unroll
    for (int k = 0; k < EPT; k++) {
        const int e = ROWS == 1 ? (lane < 63 ? (t >> 6) * 21 + lane / 3 : 1 << 20) : k * kResNT + t;
        int c = 0, p = e;
#pragma unroll
        for (int x = 0; x + 1 < C; x++)
            if (e >= end[x]) { c = x + 1; p = e - end[x]; }
        const bool valid = e < end[C - 1];
        int i, j;
        if constexpr (NB == 21) {
            const int f = first3(c % 3, ci0), m = (ci1 - f + 2) / 3 > 0 ? (ci1 - f + 2) / 3 : 1;
            i = f + 3 * (p % m);
            j = first3(c / 3, cj0) + 3 * (p / m);
        } else {
            int jr = p / cw * C, rem = p % cw;
#pragma unroll
            for (int x = 0; x + 1 < C; x++) {
                const int m = (cw - first(c, jr) + C - 1) / C;
                if (rem >= m) { rem -= m; jr++; }
                else break;
            }
            i = ci0 + first(c, jr) + C * rem;
            j = cj0 + jr;
        }
        const bool own = valid && i >= i0 && i < i1 && j >= j0 && j < j1;
        const bool read = own && ((i0 > 0 && i - i0 < hd) || (i1 < nx && i1 - 1 - i < hd) || (j0 > 0 && j - j0 < hd) ||
                                  (j1 < ny && j1 - 1 - j < hd));
        flags[k] = (valid ? c + 1 : 0) | (own ? 16 : 0) | (read ? 32 : 0);
        q[k] = valid ? (j - dj0) * ld + (i - di0) : 0;
        if (valid) {
            const long long cc = perm2d_of<C>(L.P, i, j);
#pragma unroll
            for (int b = 1; b < NB; b++) {
                const int pi = i + stencil_dx(NB, b), pj = j + stencil_dy(NB, b);
                const bool ok = pi >= 0 && pi < nx && pj >= 0 && pj < ny;
#pragma unroll
                for (int x = 0; x < 3 * ROWS; x++) Jb[k][b][x] = ok ? (HT)mg[L.J + (b * 9 + 3 * row + x) * n + cc] : (HT)0.0;
            }
#pragma unroll
            for (int x = 0; x < 3 * ROWS; x++) Di[k][x] = (HT)mg[L.Dinv + (3 * row + x) * n + cc];
#pragma unroll
            for (int x = 0; x < ROWS; x++) rh[k][x] = (HT)mg[L.rhs + (row + x) * n + cc];
        } else {
#pragma unroll
            for (int b = 1; b < NB; b++)
#pragma unroll
                for (int x = 0; x < 3 * ROWS; x++) Jb[k][b][x] = (HT)0.0;
#pragma unroll
            for (int x = 0; x < 3 * ROWS; x++) Di[k][x] = (HT)0.0;
#pragma unroll
            for (int x = 0; x < ROWS; x++) rh[k][x] = (HT)0.0;
        }
    }

    // the halo cells the thread fetches (none where one workgroup has the level): the bands below and above, then left and right
    const int below = j0 - dj0, above = dj1 - j1, left = i0 - di0, side = left + (di1 - i1);
    const int nh = (below + above) * dw + (j1 - j0) * side;
    int hq[kResHalo], hcell[kResHalo];           // hq: place in LDS | colour + 1 << 16 (0: nothing to fetch)
#pragma unroll
    for (int k = 0; k < kResHalo; k++) {
        const int e = k * kResNT + t;
        int i = 0, j = 0;
        if (e < (below + above) * dw) {
            const int r = e / dw;
            i = di0 + e - r * dw;
            j = r < below ? dj0 + r : j1 + (r - below);
        } else if (e < nh) {
            const int f = e - (below + above) * dw, r = f / side, s = f - r * side;
            j = j0 + r;
            i = s < left ? di0 + s : i1 + (s - left);
        }
        // a pass of a cross stencil moves information R cells along one axis: m passes read no cell
        // farther out (with the full stencil, every cell of the halo)
        const int ox = i < i0 ? i0 - i : (i >= i1 ? i - i1 + 1 : 0), oy = j < j0 ? j0 - j : (j >= j1 ? j - j1 + 1 : 0);
        const bool read = e < nh && (NB == 21 || (ox + R - 1) / R + (oy + R - 1) / R <= A.m);
        hq[k] = read ? ((j - dj0) * ld + (i - di0)) | ((i + j) % C + 1) << 16 : 0;
        hcell[k] = read ? j * nx + i : 0;
    }

    // dU of the tile and its halo
    for (int e = t; e < kResPL; e += kResNT) sz[e] = Cell{};
    __syncthreads();
    for (int e = t; e < dw * dh; e += kResNT) {
        const int r = e / dw, i = di0 + e - r * dw, j = dj0 + r;
        const long long fc = perm2d_of<C>(L.P, i, j);
        const long long pc = A.prolong ? perm2d_of<2>(A.Lc.P, i >> 1, j >> 1) : 0;
#pragma unroll
        for (int c = 0; c < 3; c++) {
            T v = mg[L.dU + c * n + fc];
            if (A.prolong) v = (T)((double)v + ld2(mg + A.Lc.dU, c * A.Lc.P.M + pc));
            su[r * ld + (i - di0)].v[c] = v;
        }
    }
    __syncthreads();
    // the rows have to be there before the first pass: a wait left to the loop would count the
    // exchange's stores too
    __builtin_amdgcn_s_waitcnt(0x0f70);          // vmcnt(0)

    // the merged colour passes: colours 0 .. C-1 .. 0 .. and so on, twice at every turn
    const int runs = A.nu > 0 ? A.nu * 4 * (C - 1) + 1 : 0;
    unsigned tag = A.tag;
    const double keep = 1.0 - A.omega;
    // one pass an exchange: only its colour's cells travel (not with nine colours, of which an edge
    // between two tiles need not hold every one)
    const bool filter = NB != 21 && A.m == 1;
    int since = 0;
    for (int s = 0; s < runs; s++) {
        const int ph = s % (2 * (C - 1));
        const int c = ph <= C - 1 ? ph : 2 * (C - 1) - ph;
        const bool twice = (c == 0 || c == C - 1) && s > 0 && s < runs - 1;
#pragma unroll
        for (int k = 0; k < EPT; k++) {
            if (colour(k) != c) continue;
#pragma unroll
            for (int x = 0; x < 3 * ROWS; x++) {
#pragma unroll
                for (int b = 1; b < NB; b++) keep_narrow(Jb[k][b][x]);
                keep_narrow(Di[k][x]);
            }
            // the values are read ahead of the products: a wavefront has its SIMD almost to itself, so
            // a read's latency is paid once (or, where the registers do not suffice, partly behind the
            // first products)
            Cell *u = su + q[k];
            T d[ROWS];
#pragma unroll
            for (int x = 0; x < ROWS; x++) d[x] = u->v[row + x];
            Cell y[NB];
            double r[ROWS];
#pragma unroll
            for (int x = 0; x < ROWS; x++) r[x] = (double)rh[k][x];
            auto read = [&](int b0, int b1) {
#pragma unroll
                for (int b = b0; b <= b1; b++) y[b] = u[stencil_dy(NB, b) * ld + stencil_dx(NB, b)];
                __builtin_amdgcn_sched_barrier(0);
            };
            auto add = [&](int b0, int b1) {
#pragma unroll
                for (int b = b0; b <= b1; b++) {
                    const double x0 = (double)y[b].v[0], x1 = (double)y[b].v[1], x2 = (double)y[b].v[2];
#pragma unroll
                    for (int x = 0; x < ROWS; x++)
                        r[x] = r[x] + ((double)Jb[k][b][x * 3 + 0] * x0 + (double)Jb[k][b][x * 3 + 1] * x1 +
                                       (double)Jb[k][b][x * 3 + 2] * x2);
                }
            };
            if constexpr (NB == 21) {
                read(1, 10);
                add(1, 5);
                __builtin_amdgcn_sched_barrier(0);
                read(11, 15);
                add(6, 10);
                __builtin_amdgcn_sched_barrier(0);
                read(16, 20);
                add(11, 20);
            } else if constexpr (NB == 9 && sizeof(HT) == 8) {
                read(1, 5);
                add(1, 3);
                __builtin_amdgcn_sched_barrier(0);
                read(6, 8);
                add(4, 8);
            } else {
                read(1, NB - 1);
                add(1, NB - 1);
            }
            double f[3];
            if constexpr (ROWS == 1) {
#pragma unroll
                for (int x = 0; x < 3; x++) f[x] = __shfl(r[0], lane - row + x, 64);
            } else {
#pragma unroll
                for (int x = 0; x < 3; x++) f[x] = r[x];
            }
#pragma unroll
            for (int x = 0; x < ROWS; x++) {
                const double tt = (double)Di[k][x * 3 + 0] * f[0] + (double)Di[k][x * 3 + 1] * f[1] + (double)Di[k][x * 3 + 2] * f[2];
                const T d1 = (T)(keep * (double)d[x] - A.omega * tt);
                const T d2 = (T)(keep * (double)d1 - A.omega * tt);
                u->v[row + x] = twice ? d2 : d1;
            }
        }
        if (SOLO) { __syncthreads(); continue; }
        since++;
        if (since < A.m && s < runs - 1) { __syncthreads(); continue; }
        since = 0;
        if (s == runs - 1 && !A.restr) break;
        tag++;
        unsigned long long *box = A.box + (long long)(tag & 1) * A.cells * NW;
#pragma unroll
        for (int k = 0; k < EPT; k++)
            if (edge(k) && (!filter || colour(k) == c)) {
                T own[ROWS];
#pragma unroll
                for (int x = 0; x < ROWS; x++) own[x] = su[q[k]].v[row + x];
#pragma unroll
                for (int x = 0; x < ROWS; x++) box_store(box + (cell_j(k) * nx + cell_i(k)), A.cells, tag, row + x, own[x]);
            }
        __syncthreads();     // every cell of the group is relaxed and read before the halo changes
        // the words of KB cells are loaded together, again until each cell's carry the tag
#pragma unroll
        for (int k0 = 0; k0 < kResHalo; k0 += KB) {
            if (k0 * kResNT >= nh) break;
            unsigned pend = 0;
#pragma unroll
            for (int k = k0; k < k0 + KB && k < kResHalo; k++)
                if (hq[k] && (!filter || hq[k] >> 16 == c + 1)) pend |= 1u << k;
            if (dead) pend = 0;
            long long t0 = 0;
            for (int spin = 0; pend; spin++) {
                unsigned long long v[KB][NW];
#pragma unroll
                for (int k = k0; k < k0 + KB && k < kResHalo; k++)
                    if (k * kResNT < nh)
#pragma unroll
                        for (int w = 0; w < NW; w++)
                            v[k - k0][w] = __hip_atomic_load(box + hcell[k] + w * A.cells, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
#pragma unroll
                for (int k = k0; k < k0 + KB && k < kResHalo; k++) {
                    if (k * kResNT >= nh || !(pend >> k & 1)) continue;
                    bool ok = true;
#pragma unroll
                    for (int w = 0; w < NW; w++) ok = ok && (unsigned)(v[k - k0][w] >> 32) == tag;
                    if (!ok) continue;
                    pend &= ~(1u << k);
#pragma unroll
                    for (int x = 0; x < 3; x++) box_value(v[k - k0], x, su[hq[k] & 0xffff].v[x]);
                }
                if ((spin & 255) == 255) {
                    const long long now = wall_clock64();
                    if (t0 == 0) t0 = now;
                    else if (now - t0 > kWaitTicks) { dead = 1; pend = 0; }
                }
            }
        }
        __syncthreads();
    }
    __syncthreads();
    const bool bad = !SOLO && dead != 0;

#pragma unroll
    for (int k = 0; k < EPT; k++) {
        if (!inside(k)) continue;
        const long long cc = perm2d_of<C>(L.P, cell_i(k), cell_j(k));
#pragma unroll
        for (int c = 0; c < ROWS; c++) mg[L.dU + (row + c) * n + cc] = bad ? (T)__builtin_nan("") : su[q[k]].v[row + c];
    }
    if (!A.restr) return;
    // eq. (24): rhs + J dU of every cell of the tile, then the sums over the children
    const int tw = i1 - i0;
    double a[EPT][ROWS];
#pragma unroll
    for (int k = 0; k < EPT; k++) {
        if (!inside(k)) continue;
        const Cell *u = su + q[k];
        const long long cc = perm2d_of<C>(L.P, cell_i(k), cell_j(k));
        const double y0 = (double)u->v[0], y1 = (double)u->v[1], y2 = (double)u->v[2];
#pragma unroll
        for (int x = 0; x < ROWS; x++)
            a[k][x] = (double)rh[k][x] + (ld2(mg + L.J, ((row + x) * 3 + 0) * n + cc) * y0 +
                                          ld2(mg + L.J, ((row + x) * 3 + 1) * n + cc) * y1 +
                                          ld2(mg + L.J, ((row + x) * 3 + 2) * n + cc) * y2);
#pragma unroll
        for (int b = 1; b < NB; b++) {
            const int o = stencil_dy(NB, b) * ld + stencil_dx(NB, b);
            const double x0 = (double)u[o].v[0], x1 = (double)u[o].v[1], x2 = (double)u[o].v[2];
#pragma unroll
            for (int x = 0; x < ROWS; x++)
                a[k][x] = a[k][x] + ((double)Jb[k][b][x * 3 + 0] * x0 + (double)Jb[k][b][x * 3 + 1] * x1 +
                                     (double)Jb[k][b][x * 3 + 2] * x2);
        }
    }
    __syncthreads();
    double *sa = lds.v;                          // [3][tile cells]
#pragma unroll
    for (int k = 0; k < EPT; k++) {
        if (!inside(k)) continue;
#pragma unroll
        for (int x = 0; x < ROWS; x++) sa[(row + x) * A.tx * A.ty + (cell_j(k) - j0) * tw + (cell_i(k) - i0)] = a[k][x];
    }
    __syncthreads();
    const int hw = tw / 2, hh = (j1 - j0) / 2;
    for (int e = t; e < hw * hh; e += kResNT) {
        const int jq = e / hw, iq = e - jq * hw;
        double a00[3], a10[3], a01[3], a11[3];
#pragma unroll
        for (int x = 0; x < 3; x++) {
            const double *p = sa + x * A.tx * A.ty + 2 * jq * tw + 2 * iq;
            a00[x] = p[0];
            a10[x] = p[1];
            a01[x] = p[tw];
            a11[x] = p[tw + 1];
        }
        restrict_store(mg, A.Lc, i0 / 2 + iq, j0 / 2 + jq, a00, a10, a01, a11);
    }
}

template <typename T, int NB, typename HT, int EPT>
__global__ void __launch_bounds__(kResNT) k_resident2d(T *mg, Resident2DArgs A)
{
    __shared__ ResLds lds;
    __shared__ int dead;
    if (A.state && !A.state->active) return;     // the same for every workgroup
    resident_level<T, NB, HT, EPT, false>(mg, A, blockIdx.x % A.gx, blockIdx.x / A.gx, lds, dead);
}

// ---- streamed smoothing of a level -----------------------------------------------------------

// A cross-stencil level too large for the registers of the chip (1024 x 512 in FP64: 352 MB of rows, 172
// MB of registers, of which rows can have two thirds) runs its phases in one cooperative launch too, a
// tile per compute unit with dU in LDS and the same exchange after every pass, and part of its rows
// held: in registers (one FP64 or two FP32 rows a thread) and kLdsRows in LDS.  The symmetric schedule
// passes over colour 1 every other time and over colours 0 and 2 every fourth, so colour 1 is held
// first, after as many cells of colours 0 and 2 as leave each of them one streamed cell a thread.  The
// rest is streamed in every pass, contiguously (its rows lie in tiles), and that is the bound: about 7.6 TB/s
// from the memory-side cache, which the streamed part fits (235 MB; all rows: 6.1-6.6 TB/s).
// 1024 x 512 FP64: 25.8 us a pass as separate launches, 14.2 so; FP32 13.6, 5.7.
constexpr int kStrCells = 2600;                  // LDS cells of a tile with a ring of two
constexpr int kLdsRows = 64;                     // colour 1 rows held in LDS
constexpr int kRowValues = 84;                   // eight off-diagonal blocks, D^{-1}, right-hand side

// how many of a colour's n[c] cells the registers hold (cap rows in all) and, of colour 1, LDS
__device__ __forceinline__ void streamed_split(const int n[3], int cap, int held[3], int &in_lds)
{
    held[0] = n[0] > kResNT ? n[0] - kResNT : 0;
    held[2] = n[2] > kResNT ? n[2] - kResNT : 0;
    if (held[0] + held[2] > cap) held[0] = held[2] = 0;
    int left = cap - held[0] - held[2];
    held[1] = n[1] < left ? n[1] : left;
    left -= held[1];
    in_lds = n[1] - held[1] < kLdsRows ? n[1] - held[1] : kLdsRows;
    const int more0 = n[0] - held[0] < left / 2 ? n[0] - held[0] : left / 2;
    held[0] += more0;
    left -= more0;
    held[2] += n[2] - held[2] < left ? n[2] - held[2] : left;
}

template <typename T, int EPT>
__global__ void __launch_bounds__(kResNT) k_streamed2d(T *mg, Resident2DArgs A)
{
    constexpr int NB = 9, C = 3, NW = BoxWords<T>::n;
    constexpr int RING = sizeof(T) == 8 ? 5 : 9;           // triples of a streamed row that registers hold
    typedef ResCell<T> Cell;
    __shared__ Cell sz[kStrCells];
    // rows in LDS, and for FP64 rows in registers their D^{-1} and right-hand sides (with them the rows
    // themselves would not stay in registers; read from memory, they are late while the rest streams)
    constexpr bool HOLD = sizeof(T) == 4;
    constexpr int POOL = kLdsRows * kRowValues + (HOLD ? 0 : 12 * kResNT);
    __shared__ double rows_lds[POOL > 3 * kStrCells ? POOL : 3 * kStrCells];
    __shared__ int dead;
    if (A.state && !A.state->active) return;     // the same for every workgroup
    T *const rows = (T *)rows_lds;               // [kRowValues][kLdsRows]
    T *const dr = rows + kLdsRows * kRowValues;  // [12][512]
    const Level2D &L = A.L;
    const int t = threadIdx.x, nx = L.nx, ny = L.ny;
    const int bi = blockIdx.x % A.gx, bj = blockIdx.x / A.gx;
    const int i0 = bi * A.tx, j0 = bj * A.ty;
    const int i1 = i0 + A.tx < nx ? i0 + A.tx : nx, j1 = j0 + A.ty < ny ? j0 + A.ty : ny;
    const int tw = i1 - i0, th = j1 - j0, ld = tw + 4;
    Cell *const su = sz + 2 * ld + 2;            // cell (i0, j0); the halo's place is there at a side, too, as zeros
    const long long n = L.P.M;
    if (t == 0) dead = 0;

    int cells[C], held[C], in_lds;
    long long row0[C];                           // where the tile's rows begin
#pragma unroll
    for (int c = 0; c < C; c++) {
        cells[c] = tile3_count(c, i0, j0, tw, th);
        row0[c] = tile3_start(L.P, c, i0, j0, th);
    }
    streamed_split(cells, EPT * kResNT, held, in_lds);
    // place in LDS of cell e of colour c, with bit 16 set where other tiles read it and bit 16 + b where
    // its neighbour of block b lies outside the grid
    auto place = [&](int c, int e) {
        int il, jr;
        tile3_cell(c, i0, j0, tw, e, il, jr);
        const bool read = (i0 > 0 && il < 2) || (i1 < nx && tw - 1 - il < 2) || (j0 > 0 && jr < 2) || (j1 < ny && th - 1 - jr < 2);
        int p = (jr * ld + il) | (read ? 1 << 16 : 0);
#pragma unroll
        for (int b = 1; b < NB; b++) {
            const int pi = i0 + il + stencil_dx(NB, b), pj = j0 + jr + stencil_dy(NB, b);
            if (pi < 0 || pi >= nx || pj < 0 || pj >= ny) p |= 1 << (16 + b);
        }
        return p;
    };
    auto slot_of = [&](int c, int e) { return (c == 0 ? row0[0] : c == 1 ? row0[1] : row0[2]) + e; };

    // rows in registers: the slots k * 512 + t take colour 1's cells, then colour 0's, then colour 2's
    T Jb[EPT][NB][9], Di[HOLD ? EPT : 1][9], rh[HOLD ? EPT : 1][3];
    int q[EPT], col[EPT];
    unsigned own_off[EPT];                       // byte offset of the cell in the level's arrays
#pragma unroll
    for (int k = 0; k < EPT; k++) {
        const int r = k * kResNT + t;
        int c = 1, e = r;
        if (e >= held[1]) { c = 0; e -= held[1]; if (e >= held[0]) { c = 2; e -= held[0]; } }
        const bool valid = e < held[c];
        col[k] = valid ? c : -1;
        q[k] = valid ? place(c, e) : 0;
        own_off[k] = valid ? (unsigned)(slot_of(c, e) * (int)sizeof(T)) : 0;
    }
    for (int e = t; e < in_lds * kRowValues; e += kResNT) {
        const int v = e / in_lds, r = e - v * in_lds;
        const long long cc = slot_of(1, held[1] + r);
        const bool out = v < 72 && (place(1, held[1] + r) >> (17 + v / 9) & 1);
        rows[v * kLdsRows + r] = out ? (T)0 : v < 72 ? mg[L.J + (v + 9) * n + cc] : (v < 81 ? mg[L.Dinv + (v - 72) * n + cc] : mg[L.rhs + (v - 81) * n + cc]);
    }
    // the thread's first streamed cell of each colour, and its row in LDS (the last threads', which
    // have no streamed cell of colour 1 while there are few)
    int sq[C], start[C];
#pragma unroll
    for (int c = 0; c < C; c++) {
        start[c] = held[c] + (c == 1 ? in_lds : 0);
        sq[c] = start[c] + t < cells[c] ? place(c, start[c] + t) : 0;
    }
    const int lr = kResNT - 1 - t;
    const int lq = lr < in_lds ? place(1, held[1] + lr) : 0;

    // the halo cell the thread fetches (at most 512: 2 x 2 rows and columns): place | colour + 1 << 16
    int hq = 0, hcell = 0;
    {
        const int dj0 = j0 - 2 > 0 ? j0 - 2 : 0, dj1 = j1 + 2 < ny ? j1 + 2 : ny;
        const int di0 = i0 - 2 > 0 ? i0 - 2 : 0, di1 = i1 + 2 < nx ? i1 + 2 : nx;
        const int below = j0 - dj0, above = dj1 - j1, left = i0 - di0, side = left + (di1 - i1);
        int i = -1, j = -1;
        if (t < (below + above) * tw) {
            const int r = t / tw;
            i = i0 + t - r * tw;
            j = r < below ? dj0 + r : j1 + (r - below);
        } else if (t < (below + above) * tw + th * side) {
            const int f = t - (below + above) * tw, r = f / side, x = f - r * side;
            j = j0 + r;
            i = x < left ? di0 + x : i1 + (x - left);
        }
        if (i >= 0) {
            hq = ((j - j0 + 2) * ld + (i - i0 + 2)) | ((i + j) % C + 1) << 16;
            hcell = j * nx + i;
        }
    }

    for (int e = t; e < (tw + 4) * (th + 4); e += kResNT) {
        const int r = e / ld, i = i0 - 2 + e - r * ld, j = j0 - 2 + r;
        Cell v = Cell{};
        if (i >= 0 && i < nx && j >= 0 && j < ny) {
            const long long fc = perm2d_of<C>(L.P, i, j);
            const long long pc = A.prolong ? perm2d_of<2>(A.Lc.P, i >> 1, j >> 1) : 0;
#pragma unroll
            for (int c = 0; c < 3; c++) {
                v.v[c] = mg[L.dU + c * n + fc];
                if (A.prolong) v.v[c] = (T)((double)v.v[c] + ld2(mg + A.Lc.dU, c * A.Lc.P.M + pc));
            }
        }
        sz[e] = v;
    }
    // value v of the arrays at `base` for the slot at byte offset `off` (the base and the stride are
    // uniform: no address registers)
    auto fetch = [&](long long base, int v, unsigned off) {
        return *(const T *)((const char *)(mg + base + v * n) + off);
    };
#pragma unroll
    for (int k = 0; k < EPT; k++) {
#pragma unroll
        for (int b = 1; b < NB; b++)
#pragma unroll
            for (int x = 0; x < 9; x++) {
                const T v = fetch(L.J, b * 9 + x, own_off[k]);
                Jb[k][b][x] = q[k] >> (16 + b) & 1 ? (T)0 : v;
            }
        if constexpr (HOLD) {
#pragma unroll
            for (int x = 0; x < 9; x++) Di[k][x] = fetch(L.Dinv, x, own_off[k]);
#pragma unroll
            for (int x = 0; x < 3; x++) rh[k][x] = fetch(L.rhs, x, own_off[k]);
        } else {
#pragma unroll
            for (int x = 0; x < 9; x++) dr[x * kResNT + t] = fetch(L.Dinv, x, own_off[k]);
#pragma unroll
            for (int x = 0; x < 3; x++) dr[(9 + x) * kResNT + t] = fetch(L.rhs, x, own_off[k]);
        }
    }
    __syncthreads();
    __builtin_amdgcn_s_waitcnt(0x0f70);          // vmcnt(0)

    const int runs = A.nu > 0 ? A.nu * 4 * (C - 1) + 1 : 0;
    const double keep = 1.0 - A.omega;
    unsigned tag = A.tag;
    for (int s = 0; s < runs; s++) {
        const int ph = s % (2 * (C - 1));
        const int c = ph <= C - 1 ? ph : 2 * (C - 1) - ph;
        const bool twice = (c == 0 || c == C - 1) && s > 0 && s < runs - 1, send = s < runs - 1 || A.restr;
        if (send) tag++;
        unsigned long long *box = A.box + (long long)(tag & 1) * A.cells * NW;
        // relax the cell at place p by D^{-1} r = tt, and publish it
        auto relax = [&](int p, const double tt[3]) {
            Cell *u = su + (p & 0xffff);
            T v[3];
#pragma unroll
            for (int x = 0; x < 3; x++) {
                const T d1 = (T)(keep * (double)u->v[x] - A.omega * tt[x]);
                const T d2 = (T)(keep * (double)d1 - A.omega * tt[x]);
                v[x] = twice ? d2 : d1;
                u->v[x] = v[x];
            }
            if (send && (p >> 16 & 1)) {
                const int il = (p & 0xffff) % ld, jr = (p & 0xffff) / ld;
#pragma unroll
                for (int x = 0; x < 3; x++) box_store(box + ((j0 + jr) * nx + i0 + il), A.cells, tag, x, v[x]);
            }
        };
        auto apply = [&](const T *D, const double r[3], double tt[3]) {
#pragma unroll
            for (int x = 0; x < 3; x++) tt[x] = (double)D[x * 3 + 0] * r[0] + (double)D[x * 3 + 1] * r[1] + (double)D[x * 3 + 2] * r[2];
        };
        auto add = [&](double r[3], const Cell &y, const T *J) {
            const double x0 = (double)y.v[0], x1 = (double)y.v[1], x2 = (double)y.v[2];
#pragma unroll
            for (int x = 0; x < 3; x++) r[x] = r[x] + ((double)J[x * 3 + 0] * x0 + (double)J[x * 3 + 1] * x1 + (double)J[x * 3 + 2] * x2);
        };
#pragma unroll
        for (int k = 0; k < EPT; k++) {
            if (col[k] != c) continue;
#pragma unroll
            for (int x = 0; x < 9; x++) {
#pragma unroll
                for (int b = 1; b < NB; b++) keep_narrow(Jb[k][b][x]);
                if constexpr (HOLD) keep_narrow(Di[k][x]);
            }
            const Cell *u = su + (q[k] & 0xffff);
            double r[3], tt[3];
#pragma unroll
            for (int x = 0; x < 3; x++) r[x] = (double)(HOLD ? rh[HOLD ? k : 0][x] : dr[(9 + x) * kResNT + t]);
#pragma unroll
            for (int b = 1; b < NB; b++) {
                if (b == 5) __builtin_amdgcn_sched_barrier(0);
                add(r, u[stencil_dy(NB, b) * ld + stencil_dx(NB, b)], Jb[k][b]);
            }
            T D[9];
#pragma unroll
            for (int x = 0; x < 9; x++) D[x] = HOLD ? Di[HOLD ? k : 0][x] : dr[x * kResNT + t];
            apply(D, r, tt);
            relax(q[k], tt);
        }
        for (int e = start[c] + t, p = sq[c]; e < cells[c];) {
            // the row as 27 triples (a row of each block, then of D^{-1}), RING - 1 of them on their way
            const unsigned off = (unsigned)(slot_of(c, e) * (int)sizeof(T));
            const Cell *u = su + (p & 0xffff);
            T v[RING][3];
            double r[3], tt[3];
            auto triple = [&](int g) {
#pragma unroll
                for (int x = 0; x < 3; x++)
                    v[g % RING][x] = g < 24 ? fetch(L.J, 9 + 3 * g + x, off) : fetch(L.Dinv, 3 * (g - 24) + x, off);
            };
#pragma unroll
            for (int x = 0; x < 3; x++) r[x] = (double)fetch(L.rhs, x, off);
#pragma unroll
            for (int g = 0; g < RING - 1; g++) triple(g);
#pragma unroll
            for (int b = 1; b < NB; b++) {
                const Cell y = u[stencil_dy(NB, b) * ld + stencil_dx(NB, b)];
                const double x0 = (double)y.v[0], x1 = (double)y.v[1], x2 = (double)y.v[2];
#pragma unroll
                for (int x = 0; x < 3; x++) {
                    const int g = (b - 1) * 3 + x;
                    if (g + RING - 1 < 27) triple(g + RING - 1);
                    __builtin_amdgcn_sched_barrier(0);
                    const T *J = v[g % RING];
                    const double a = (double)J[0] * x0 + (double)J[1] * x1 + (double)J[2] * x2;
                    if (!(p >> (16 + b) & 1)) r[x] = r[x] + a;
                }
            }
#pragma unroll
            for (int x = 0; x < 3; x++) {
                const T *D = v[(24 + x) % RING];
                tt[x] = (double)D[0] * r[0] + (double)D[1] * r[1] + (double)D[2] * r[2];
            }
            relax(p, tt);
            e += kResNT;
            if (e < cells[c]) p = place(c, e);
        }
        if (c == 1 && lr < in_lds) {
            const Cell *u = su + (lq & 0xffff);
            double r[3];
#pragma unroll
            for (int x = 0; x < 3; x++) r[x] = (double)rows[(81 + x) * kLdsRows + lr];
            T D[9];
#pragma unroll
            for (int b = 1; b < NB; b++) {
                T J[9];
#pragma unroll
                for (int x = 0; x < 9; x++) J[x] = rows[((b - 1) * 9 + x) * kLdsRows + lr];
                if (b & 1) __builtin_amdgcn_sched_barrier(0);    // two blocks at a time: the registers are full
                add(r, u[stencil_dy(NB, b) * ld + stencil_dx(NB, b)], J);
            }
#pragma unroll
            for (int x = 0; x < 9; x++) D[x] = rows[(72 + x) * kLdsRows + lr];
            double tt[3];
            apply(D, r, tt);
            relax(lq, tt);
        }
        if (!send) break;
        __syncthreads();
        if (hq >> 16 == c + 1 && !dead) {
            long long t0 = 0;
            for (int spin = 0;; spin++) {
                unsigned long long v[NW];
                bool ok = true;
#pragma unroll
                for (int w = 0; w < NW; w++) v[w] = __hip_atomic_load(box + hcell + w * A.cells, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
#pragma unroll
                for (int w = 0; w < NW; w++) ok = ok && (unsigned)(v[w] >> 32) == tag;
                if (ok) {
#pragma unroll
                    for (int x = 0; x < 3; x++) box_value(v, x, sz[hq & 0xffff].v[x]);
                    break;
                }
                if ((spin & 255) == 255) {
                    const long long now = wall_clock64();
                    if (t0 == 0) t0 = now;
                    else if (now - t0 > kWaitTicks) { dead = 1; break; }
                }
            }
        }
        __syncthreads();
    }
    __syncthreads();
    const bool bad = dead != 0;

    // dU of the tile's cells and, for eq. (24), rhs + J dU (rows read from memory once more)
    double *sa = rows_lds;                       // [3][tile cells]
#pragma unroll 1
    for (int c = 0; c < C; c++)
        for (int e = t; e < cells[c]; e += kResNT) {
            const int f = place(c, e), p = f & 0xffff, il = p % ld, jr = p / ld;
            const long long cc = slot_of(c, e), uc = perm2d_of<C>(L.P, i0 + il, j0 + jr);
            const Cell *u = su + p;
#pragma unroll
            for (int x = 0; x < 3; x++) mg[L.dU + x * n + uc] = bad ? (T)__builtin_nan("") : u->v[x];
            if (!A.restr) continue;
            double a[3];
#pragma unroll
            for (int x = 0; x < 3; x++) a[x] = (double)mg[L.rhs + x * n + cc];
            T v[2][9];
#pragma unroll
            for (int x = 0; x < 9; x++) v[0][x] = mg[L.J + x * n + cc];
#pragma unroll
            for (int b = 0; b < NB; b++) {
                if (b + 1 < NB) {
#pragma unroll
                    for (int x = 0; x < 9; x++) v[(b + 1) & 1][x] = mg[L.J + ((b + 1) * 9 + x) * n + cc];
                }
                __builtin_amdgcn_sched_barrier(0);
                const Cell y = u[stencil_dy(NB, b) * ld + stencil_dx(NB, b)];
                const double x0 = (double)y.v[0], x1 = (double)y.v[1], x2 = (double)y.v[2];
#pragma unroll
                for (int x = 0; x < 3; x++) {
                    const double w = (double)v[b & 1][x * 3 + 0] * x0 + (double)v[b & 1][x * 3 + 1] * x1 + (double)v[b & 1][x * 3 + 2] * x2;
                    if (b == 0 || !(f >> (16 + b) & 1)) a[x] = a[x] + w;
                }
            }
#pragma unroll
            for (int x = 0; x < 3; x++) sa[x * tw * th + jr * tw + il] = a[x];
        }
    if (!A.restr) return;
    __syncthreads();
    const int hw = tw / 2, hh = th / 2;
    for (int e = t; e < hw * hh; e += kResNT) {
        const int jq = e / hw, iq = e - jq * hw;
        double a00[3], a10[3], a01[3], a11[3];
#pragma unroll
        for (int x = 0; x < 3; x++) {
            const double *p = sa + x * tw * th + 2 * jq * tw + 2 * iq;
            a00[x] = p[0];
            a10[x] = p[1];
            a01[x] = p[tw];
            a11[x] = p[tw + 1];
        }
        restrict_store(mg, A.Lc, i0 / 2 + iq, j0 / 2 + jq, a00, a10, a01, a11);
    }
}

// Coarsest level: Gaussian elimination with partial pivoting of the dense system sum J dU = -rhs
// (unknown (j*nx + i)*3 + c), split into a factorisation done once per operator and a solve per
// V-cycle.  The factorisation takes the pivots and eliminates exactly as the plain algorithm does
// (largest magnitude, first on ties; rows with a zero multiplier untouched) and keeps, in the
// workspace, the eliminated matrix with each multiplier in the place it eliminates (rows
// interchanged whole, multipliers included) and the row permutation.  The solve then applies the
// permutation to the right-hand side, the multipliers column by column (the same operations on
// the same values as eliminating the right-hand side alongside), and back substitution.
//
// Both are chains of M <= 120 dependent steps, bound by what one step costs.  The factorisation keeps
// the matrix in registers (lane l of wavefront w has rows l and l + 64 of the columns w, w + 16, ...),
// so a step is the owning wavefront's pivot search and multipliers, one barrier, and every
// wavefront's update (270 -> 104 us at M = 96, before with the matrix in LDS and five barriers a step).  Rows
// are interchanged by number only.  The solve runs in one wavefront with x in registers, without
// barriers.
struct CoarseLU {
    double *A;    // [M][M], column-major, rows in pivot order
    int *perm;    // [M]: the row's place before the interchanges + (its last nonzero column << 16)
};

__device__ __forceinline__ CoarseLU coarse_lu(double *base, int M) { return CoarseLU{base, (int *)(base + (long long)M * M)}; }

__device__ __forceinline__ double lane_value(double v, int lane)
{
    const unsigned long long b = (unsigned long long)__double_as_longlong(v);
    const unsigned lo = (unsigned)__builtin_amdgcn_readlane((int)(unsigned)b, lane);
    const unsigned hi = (unsigned)__builtin_amdgcn_readlane((int)(unsigned)(b >> 32), lane);
    return __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}

// max of v and the value CTRL lanes over (a DPP move); lanes without a source keep v
template <int CTRL>
__device__ __forceinline__ double dpp_max(double v)
{
    const unsigned long long b = (unsigned long long)__double_as_longlong(v);
    const int lo = (int)(unsigned)b, hi = (int)(unsigned)(b >> 32);
    const unsigned l2 = (unsigned)__builtin_amdgcn_update_dpp(lo, lo, CTRL, 0xf, 0xf, false);
    const unsigned h2 = (unsigned)__builtin_amdgcn_update_dpp(hi, hi, CTRL, 0xf, 0xf, false);
    const double w = __longlong_as_double((long long)(((unsigned long long)h2 << 32) | l2));
    return w > v ? w : v;
}

// the largest v of the wavefront (no NaN among them)
__device__ __forceinline__ double wave_max(double v)
{
    v = dpp_max<0x111>(v);   // row_shr 1, 2, 4, 8: lane 15 of each row of 16 has the row's maximum
    v = dpp_max<0x112>(v);
    v = dpp_max<0x114>(v);
    v = dpp_max<0x118>(v);
    return fmax(fmax(lane_value(v, 15), lane_value(v, 31)), fmax(lane_value(v, 47), lane_value(v, 63)));
}

template <typename T>
__global__ void __launch_bounds__(1024) k_coarse_factor2d(T *mg, Level2D L, double *lu_base)
{
    constexpr int MM = 3 * kMaxCoarse2D, NW = 16, NQ = (MM + NW - 1) / NW;
    static_assert(MM <= 128, "two rows a lane");
    __shared__ double A[MM * MM];
    __shared__ double fcol[2][128];
    __shared__ int piv[2][2];            // the pivot row and its place
    const int nx = L.nx, ny = L.ny, n = nx * ny, M = 3 * n;
    const long long Ms = L.P.M;
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
    for (int e = t; e < M * M; e += 1024) A[e] = 0.0;
    __syncthreads();
    for (int e = t; e < n * L.nb * 9; e += 1024) {
        const int cell = e % n, be = e / n, b = be / 9, rc = be - 9 * b;
        const int i = cell % nx, j = cell / nx;
        int di, dj;
        stencil_off(L.nb, b, di, dj);
        const int pi = i + di, pj = j + dj;
        if (pi < 0 || pi >= nx || pj < 0 || pj >= ny) continue;
        A[((pj * nx + pi) * 3 + rc % 3) * M + cell * 3 + rc / 3] = ld2(mg + L.J, (long long)be * Ms + perm2d(L.P, i, j));
    }
    __syncthreads();
    double a[NQ][2];
#pragma unroll
    for (int q = 0; q < NQ; q++) {
        const int c = wave + NW * q;
        a[q][0] = c < M && lane < M ? A[c * M + lane] : 0.0;
        a[q][1] = c < M && lane + 64 < M ? A[c * M + lane + 64] : 0.0;
    }
    // the place of rows lane and lane + 64; rows past the matrix stay behind every k
    int p0 = lane < M ? lane : -1, p1 = lane + 64 < M ? lane + 64 : -1;
#pragma unroll
    for (int q = 0; q < NQ; q++) {
        for (int w = 0; w < NW; w++) {
            const int k = q * NW + w, buf = k & 1;
            if (k >= M) break;
            if (wave == w) {
                // pivot: the largest magnitude at a place >= k, the first place on ties, place k if no
                // entry compares
                const double m0 = fabs(a[q][0]), m1 = fabs(a[q][1]);
                const double v0 = p0 >= k && m0 >= 0.0 ? m0 : -1.0, v1 = p1 >= k && m1 >= 0.0 ? m1 : -1.0;
                const double top = wave_max(v0 > v1 ? v0 : v1);
                unsigned long long t0 = __ballot(top < 0.0 ? p0 == k : v0 == top), t1 = __ballot(top < 0.0 ? p1 == k : v1 == top);
                int row = t0 ? __builtin_ctzll(t0) : 64 + __builtin_ctzll(t1);
                int place = row < 64 ? __builtin_amdgcn_readlane(p0, row) : __builtin_amdgcn_readlane(p1, row - 64);
                if (__popcll(t0) + __popcll(t1) > 1) {
                    for (; t0; t0 &= t0 - 1) {
                        const int r = __builtin_ctzll(t0), pl = __builtin_amdgcn_readlane(p0, r);
                        if (pl < place) { place = pl; row = r; }
                    }
                    for (; t1; t1 &= t1 - 1) {
                        const int r = __builtin_ctzll(t1), pl = __builtin_amdgcn_readlane(p1, r);
                        if (pl < place) { place = pl; row = r + 64; }
                    }
                }
                const double akk = row < 64 ? lane_value(a[q][0], row) : lane_value(a[q][1], row - 64);
                double f0 = 0.0, f1 = 0.0;
                if (p0 >= k && lane != row) a[q][0] = f0 = a[q][0] / akk;
                if (p1 >= k && lane + 64 != row) a[q][1] = f1 = a[q][1] / akk;
                fcol[buf][lane] = f0;
                fcol[buf][lane + 64] = f1;
                if (lane == 0) { piv[buf][0] = row; piv[buf][1] = place; }
            }
            __syncthreads();     // the other buffer is free again: every wavefront has passed its step
            const int row = __builtin_amdgcn_readfirstlane(piv[buf][0]), place = __builtin_amdgcn_readfirstlane(piv[buf][1]);
            const double f0 = fcol[buf][lane], f1 = fcol[buf][lane + 64];
            if (p0 == k) p0 = place;
            if (p1 == k) p1 = place;
            if (lane == row) p0 = k;
            if (lane + 64 == row) p1 = k;
#pragma unroll
            for (int x = q; x < NQ; x++) {
                if (wave + NW * x <= k) continue;
                const double u = row < 64 ? lane_value(a[x][0], row) : lane_value(a[x][1], row - 64);
                if (f0 != 0.0) a[x][0] -= f0 * u;
                if (f1 != 0.0) a[x][1] -= f1 * u;
            }
        }
    }
    const CoarseLU lu = coarse_lu(lu_base, M);
    __shared__ int ext[MM];
    for (int r = t; r < M; r += 1024) ext[r] = r;
    __syncthreads();
#pragma unroll
    for (int q = 0; q < NQ; q++) {
        const int c = wave + NW * q;
        if (c >= M) continue;
        if (p0 >= 0) {
            lu.A[c * M + p0] = a[q][0];
            if (a[q][0] != 0.0) atomicMax(&ext[p0], c);
        }
        if (p1 >= 0) {
            lu.A[c * M + p1] = a[q][1];
            if (a[q][1] != 0.0) atomicMax(&ext[p1], c);
        }
    }
    __syncthreads();
    if (wave == 0) {
        if (p0 >= 0) lu.perm[p0] = lane | ext[p0] << 16;
        if (p1 >= 0) lu.perm[p1] = (lane + 64) | ext[p1] << 16;
    }
}

// solve with the factors of k_coarse_factor2d; A ([M][M + 1]) and sum ([144]) are LDS arrays of the
// calling workgroup of 512 threads
template <typename T>
__device__ __forceinline__ void coarse_apply(T *mg, const Level2D &L, const double *lu_base, double *A, double *sum)
{
    constexpr int NC = (3 * kMaxCoarse2D + 7) / 8;
    const int nx = L.nx, n = nx * L.ny, M = 3 * n, ld = M + 1;
    const long long Ms = L.P.M;
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
    const CoarseLU lu = coarse_lu(const_cast<double *>(lu_base), M);
    {
        double v[NC][2];
#pragma unroll
        for (int q = 0; q < NC; q++) {
            const int c = wave + 8 * q;
            v[q][0] = c < M && lane < M ? lu.A[c * M + lane] : 0.0;
            v[q][1] = c < M && lane + 64 < M ? lu.A[c * M + lane + 64] : 0.0;
        }
#pragma unroll
        for (int q = 0; q < NC; q++) {
            const int c = wave + 8 * q;
            if (c < M && lane < M) A[c * ld + lane] = v[q][0];
            if (c < M && lane + 64 < M) A[c * ld + lane + 64] = v[q][1];
        }
    }
    if (t < 144) sum[t] = 0.0;
    __syncthreads();
    if (t < 64) {
        // x of rows t and t + 64 (in pivot order) in registers
        const int i0 = t < M ? lu.perm[t] : 0, i1 = t + 64 < M ? lu.perm[t + 64] : 0;
        auto load = [&](int src) { const int cell = src / 3; return -ld2(mg + L.rhs, (src % 3) * Ms + perm2d(L.P, cell % nx, cell / nx)); };
        double x0 = t < M ? load(i0 & 0xffff) : 0.0, x1 = t + 64 < M ? load(i1 & 0xffff) : 0.0;
        // rows t and t + 64 of column k, 0 where the row is not below the diagonal
        auto below = [&](int k, double &f0, double &f1) {
            f0 = t > k && t < M ? A[k * ld + t] : 0.0;
            f1 = t + 64 > k && t + 64 < M ? A[k * ld + t + 64] : 0.0;
        };
        double f0, f1;
        below(0, f0, f1);
        for (int k = 0; k < M - 1; k++) {
            double g0, g1;
            below(k + 1, g0, g1);
            const double xk = k < 64 ? lane_value(x0, k) : lane_value(x1, k - 64);
            x0 = f0 != 0.0 ? x0 - f0 * xk : x0;
            x1 = f1 != 0.0 ? x1 - f1 * xk : x1;
            f0 = g0;
            f1 = g1;
        }
        // back substitution row by row, each row's sum over the later unknowns in ascending column
        // order (the order of a plain dense solve, so the result rounds like one): the products in
        // parallel, through LDS, their sum a chain that ends at the row's last nonzero
        auto row = [&](int k, double &u0, double &u1, double &akk) {
            u0 = t < M ? A[t * ld + k] : 0.0;
            u1 = t + 64 < M ? A[(t + 64) * ld + k] : 0.0;
            akk = A[k * ld + k];
        };
        double u0, u1, akk;
        row(M - 1, u0, u1, akk);
        for (int k = M - 1; k >= 0; k--) {
            const int last = (k < 64 ? __builtin_amdgcn_readlane(i0, k) : __builtin_amdgcn_readlane(i1, k - 64)) >> 16;
            sum[t] = t > k && t <= last ? u0 * x0 : 0.0;
            sum[t + 64] = t + 64 > k && t + 64 <= last ? u1 * x1 : 0.0;
            __builtin_amdgcn_wave_barrier();
            double s = k < 64 ? lane_value(x0, k) : lane_value(x1, k - 64);
            const double a = akk;
            row(k > 0 ? k - 1 : 0, u0, u1, akk);
            for (int c = (k + 1) & ~1; c <= last; c += 8) {      // zeros before the first and after the last term
                double2 p[4];
#pragma unroll
                for (int q = 0; q < 4; q++) p[q] = *(const double2 *)(sum + c + 2 * q);
#pragma unroll
                for (int q = 0; q < 4; q++) {
                    s -= p[q].x;
                    s -= p[q].y;
                }
            }
            __builtin_amdgcn_wave_barrier();
            s = s / a;
            if (t == k) x0 = s;
            if (t + 64 == k) x1 = s;
        }
        auto store = [&](int r, double v) { const int cell = r / 3; mg[L.dU + (r % 3) * Ms + perm2d(L.P, cell % nx, cell / nx)] = (T)v; };
        if (t < M) store(t, x0);
        if (t + 64 < M) store(t + 64, x1);
    }
    __syncthreads();
}

// The bottom of a V-cycle in one workgroup: from level `first` (a small level) down to the
// coarsest and back, with every pass of Algorithm 2 on those levels (the same schedule of merged
// colour passes as the launches on the finer levels) separated by workgroup barriers instead of
// kernel boundaries.  Used for levels of at most kBottom2DCells cells, where a launch costs more
// than the pass itself.
struct Bottom2DArgs {
    Level2D L[kMaxLevels];
    int first, levels, nu1, nu2;
    double omega;
    const double *lu;
    int sweeps;          // smoother: 0 the multicolour schedule, 1 the directional sweeps D1-D4
};

// NBF: the stencil of the bottom's first level (the finest level when the whole hierarchy fits
// one workgroup, else a five-point level); the levels below it have five points.  Only the
// passes a launch can meet are compiled into it.  The five-point and cross levels (at most 512
// cells: one a thread) keep their rows in registers (resident_level); the 21-cell level and the
// directional sweeps read them in every pass.
template <typename T, int NBF>
__device__ __forceinline__ void bottom_smooth(T *mg, const Level2D &L, int nu, double omega, int sweeps)
{
    if (sweeps) {
        if (NBF != 5 && L.nb == NBF) sweeps_level<T, NBF>(mg, L, nu, omega);
        else sweeps_level<T, 5>(mg, L, nu, omega);
        return;
    }
    if constexpr (NBF == 21) {
        const long long slots = (long long)L.P.ny * L.P.W;
        int cur = -1, run = 0;
        for (int it = 0; it <= nu; it++) {
            for (int half = 0; half < 4; half++)
                for (int q = 0; q < 9; q++) {
                    const bool last = it == nu;
                    const int c = (half & 1) ? 8 - q : q;
                    if (!last && c == cur) { run++; continue; }
                    if (run > 0) {
                        for (long long p = threadIdx.x; p < slots; p += blockDim.x) smooth_slot<T, 21>(mg, L, cur, omega, run, p);
                        __syncthreads();
                    }
                    if (last) return;
                    cur = c;
                    run = 1;
                }
        }
    }
}

template <typename T, int NBF>
__global__ void __launch_bounds__(512) k_bottom2d(T *mg, Bottom2DArgs B)
{
    constexpr int MM = 3 * kMaxCoarse2D;
    __shared__ double A[MM * (MM + 1)];
    __shared__ __align__(16) double sum[144];
    __shared__ ResLds lds;
    const int last = B.levels - 1;
    Resident2DArgs R;
    R.m = 1;
    R.omega = B.omega;
    int dead = 0;
    // a phase of level l with the rows in registers; false: the level is not of that kind
    auto phase = [&](int l, int nu, int prolong, int restr) {
        const Level2D &L = B.L[l];
        if (B.sweeps || L.nb == 21 || (long long)L.nx * L.ny > kResNT) return false;
        R.L = L;
        R.Lc = B.L[l + 1];
        R.tx = L.nx;
        R.ty = L.ny;
        R.nu = nu;
        R.prolong = prolong;
        R.restr = restr;
        if (NBF == 9 && L.nb == 9) resident_level<T, 9, double, 1, true>(mg, R, 0, 0, lds, dead);
        else resident_level<T, 5, double, 1, true>(mg, R, 0, 0, lds, dead);
        __syncthreads();
        return true;
    };
    for (int l = B.first; l < last; l++) {
        if (phase(l, B.nu1, 0, 1)) continue;
        bottom_smooth<T, NBF>(mg, B.L[l], B.nu1, B.omega, B.sweeps);
        const Level2D &Lc = B.L[l + 1];
        for (int e = threadIdx.x; e < Lc.nx * Lc.ny; e += blockDim.x) restrict_cell(mg, B.L[l], Lc, e % Lc.nx, e / Lc.nx);
        __syncthreads();
    }
    coarse_apply(mg, B.L[last], B.lu, A, sum);
    __syncthreads();
    for (int l = last - 1; l >= B.first; l--) {
        if (phase(l, B.nu2, 1, 0)) continue;
        const Level2D &Lf = B.L[l];
        for (int e = threadIdx.x; e < Lf.nx * Lf.ny; e += blockDim.x) prolong_cell(mg, Lf, B.L[l + 1], e % Lf.nx, e / Lf.nx);
        __syncthreads();
        bottom_smooth<T, NBF>(mg, Lf, B.nu2, B.omega, B.sweeps);
    }
}

// inverse of the centre blocks of an FP64 level-0 operator in the natural order ([nb*9][n],
// block 0 first), written in the level's order
template <typename T>
__global__ void k_dinv2d(const double *J, T *Dinv, Level2D L0)
{
    const long long n = (long long)L0.nx * L0.ny;
    for (long long c = blockIdx.x * (long long)blockDim.x + threadIdx.x; c < n; c += (long long)gridDim.x * blockDim.x) {
        double D[9], B[9];
#pragma unroll
        for (int e = 0; e < 9; e++) D[e] = J[e * n + c];
        inv3d(D, B);
        const long long q = perm2d_rows(L0.P, (int)(c % L0.nx), (int)(c / L0.nx));
#pragma unroll
        for (int e = 0; e < 9; e++) Dinv[e * L0.P.M + q] = (T)B[e];
    }
}

// per-cell entries between the natural order [nent][n] and a level's order [nent][M], of rows (J, rhs)
// or of dU
template <typename S, typename D>
__global__ void k_permute2d(const S *src, D *dst, Level2D L, int nent, int rows, int to_level)
{
    const long long n = (long long)L.nx * L.ny, total = n * nent;
    for (long long e = blockIdx.x * (long long)blockDim.x + threadIdx.x; e < total; e += (long long)gridDim.x * blockDim.x) {
        const long long c = e % n, a = e / n;
        const int i = (int)(c % L.nx), j = (int)(c / L.nx);
        const long long q = rows ? perm2d_rows(L.P, i, j) : perm2d(L.P, i, j);
        if (to_level) dst[a * L.P.M + q] = (D)src[e];
        else dst[e] = (D)src[a * L.P.M + q];
    }
}

template <typename T>
__global__ void k_fill(T *p, long long n)
{
    for (long long i = blockIdx.x * (long long)blockDim.x + threadIdx.x; i < n; i += (long long)gridDim.x * blockDim.x)
        p[i] = (T)0.0;
}

// eq. (14): U <- U + tau dU (skipped once the Newton iteration has stopped); U in the natural
// order [3][ny][nx]
template <typename T>
__global__ void k_update2d(double *U, const T *mg, Level2D L0, double tau, const NewtonState *S)
{
    if (S && !S->active) return;
    const long long n = (long long)L0.nx * L0.ny;
    for (long long e = blockIdx.x * (long long)blockDim.x + threadIdx.x; e < 3 * n; e += (long long)gridDim.x * blockDim.x) {
        const long long c = e % n, comp = e / n;
        const long long q = perm2d(L0.P, (int)(c % L0.nx), (int)(c / L0.nx));
        U[e] = U[e] + tau * ld2(mg + L0.dU, comp * L0.P.M + q);
    }
}

// res from the tile partials, Newton counter and stopping test (Algorithm 1)
__global__ void __launch_bounds__(256) k_state2d(const double *partial, int ntiles, long long ncells, double tol,
                                                 int n_max, NewtonState *S, double *hist, int max_hist, int init)
{
    __shared__ double red[4];
    double v = 0.0;
    for (int k = threadIdx.x; k < ntiles; k += 256) v += partial[k];
    for (int off = 32; off > 0; off >>= 1) v += __shfl_down(v, off, 64);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
    __syncthreads();
    if (threadIdx.x != 0) return;
    const double res = (red[0] + red[1] + red[2] + red[3]) / (double)ncells;
    if (init) {
        S->res = res; S->n = 0; S->active = 1; S->status = NMG_NOT_CONVERGED;
        if (!(res == res) || res > 1e300) { S->active = 0; S->status = NMG_ENONFINITE; }
        return;
    }
    if (!S->active) return;
    S->res = res;
    if (hist && S->n < max_hist) hist[S->n] = res;
    S->n += 1;
    if (!(res == res) || res > 1e300) { S->active = 0; S->status = NMG_ENONFINITE; }
    else if (res < tol) { S->active = 0; S->status = NMG_OK; }
    else if (S->n >= n_max) { S->active = 0; S->status = NMG_NOT_CONVERGED; }
}

// ---- nested iteration: Appendix A in two dimensions (eq. A.3) ------------------------------

// Eq. (A.2) from three consecutive coarse values um, u0, up of a line centred at cell k, for
// half h (0 or 1) of coarse cell j: in the interior j = k and the half's average of the quadratic
// (A.1) has the weights (1/8, 1, -1/8) or (-1/8, 1, 1/8); the first and last cell of the line
// (j = 0, k = 1 or j = n-1, k = n-2) average the quadratic centred one cell inward over their
// half.
__device__ __forceinline__ double a2_from3(double um, double u0, double up, int j, int k, int h)
{
    if (j == k) {
        if (h == 0) return um / 8.0 + u0 - up / 8.0;
        return -um / 8.0 + u0 + up / 8.0;
    }
    const double a = (up - um) / 2.0;
    const double b = (um - 2.0 * u0 + up) / 2.0;
    const double lo = (double)(j - k) - 0.5 + 0.5 * h, hi = lo + 0.5;
    const double m1 = (lo + hi) / 2.0;                      // mean of xi over the half
    const double m2 = (lo * lo + lo * hi + hi * hi) / 3.0;  // mean of xi^2
    return u0 + a * m1 + b * (m2 - 1.0 / 12.0);
}

__device__ __forceinline__ int a2_centre(int j, int n) { return j >= 1 && j <= n - 2 ? j : (j == 0 ? 1 : n - 2); }

// Fine cell (fi, fj) of component c: the polynomial of eq. (A.3) is the tensor product of the
// quadratics (A.1), so its average over a quarter of a coarse cell is eq. (A.2) along x in the
// three coarse rows it needs, then eq. (A.2) along y of those three values (the same operations
// in the same order as refining every coarse row in x first and every fine column in y after).
__global__ void __launch_bounds__(256) k_interp_a3(const double *Uc, int nxc, int nyc, double *Uf)
{
    const int fi = blockIdx.x * blockDim.x + threadIdx.x, fj = blockIdx.y, c = blockIdx.z;
    const int nxf = 2 * nxc;
    if (fi >= nxf) return;
    const double *u = Uc + (long long)c * nyc * nxc;
    const int ic = fi >> 1, hx = fi & 1, jc = fj >> 1, hy = fj & 1;
    const int kx = a2_centre(ic, nxc), ky = a2_centre(jc, nyc);
    double t[3];
#pragma unroll
    for (int q = 0; q < 3; q++) {
        const double *row = u + (long long)(ky - 1 + q) * nxc;
        t[q] = a2_from3(row[kx - 1], row[kx], row[kx + 1], ic, kx, hx);
    }
    Uf[((long long)c * 2 * nyc + fj) * nxf + fi] = a2_from3(t[0], t[1], t[2], jc, ky, hy);
}

hipError_t launch_interp_a3(const double *Uc, int nxc, int nyc, double *Uf, hipStream_t s)
{
    if (nxc < 3 || nyc < 3 || 2 * (long long)nyc > 65535) return hipErrorInvalidValue;   // grid.y holds the fine rows
    dim3 grid((2 * nxc + 255) / 256, 2 * nyc, 3);
    hipLaunchKernelGGL(k_interp_a3, grid, dim3(256), 0, s, Uc, nxc, nyc, Uf);
    return hipGetLastError();
}

// ---- launchers ---------------------------------------------------------------------------

#define DISPATCH(prec, KER, grid, block, ...)                                                      \
    do {                                                                                           \
        if ((prec) == NMG_FP32_MG) hipLaunchKernelGGL(KER<float>, grid, block, 0, s, (float *)mg, __VA_ARGS__); \
        else hipLaunchKernelGGL(KER<double>, grid, block, 0, s, (double *)mg, __VA_ARGS__);       \
    } while (0)

hipError_t launch_coarsen2d(void *mg, const Level2D &Lf, const Level2D &Lc, int prec, hipStream_t s)
{
    const dim3 grid((Lc.nx + 63) / 64, Lc.ny, 5);
    const bool f32 = prec == NMG_FP32_MG;
    float *mf = (float *)mg;
    double *md = (double *)mg;
    if (Lf.nb == 21) {
        if (f32) hipLaunchKernelGGL((k_coarsen2d<float, 21>), grid, dim3(64), 0, s, mf, Lf, Lc);
        else hipLaunchKernelGGL((k_coarsen2d<double, 21>), grid, dim3(64), 0, s, md, Lf, Lc);
    } else if (Lf.nb == 9) {
        if (f32) hipLaunchKernelGGL((k_coarsen2d<float, 9>), grid, dim3(64), 0, s, mf, Lf, Lc);
        else hipLaunchKernelGGL((k_coarsen2d<double, 9>), grid, dim3(64), 0, s, md, Lf, Lc);
    } else {
        if (f32) hipLaunchKernelGGL((k_coarsen2d<float, 5>), grid, dim3(64), 0, s, mf, Lf, Lc);
        else hipLaunchKernelGGL((k_coarsen2d<double, 5>), grid, dim3(64), 0, s, md, Lf, Lc);
    }
    return hipGetLastError();
}

// The full stencil's passes take the three-lanes-per-cell form: a colour holds a ninth of the
// cells, too few for one thread per cell to fill the chip, and a cell's 20 off-diagonal blocks
// are a long chain of loads for one thread (measured on the 1024 x 512 wedge: 35 against 56 ms
// per FP64 V-cycle, 30 against 62 ms in FP32).  The cross and five-point passes keep one thread
// per cell, whose loads all issue up front (13.2 against 13.7 ms FP64, 8.3 against 10.8 ms FP32
// per J9 V-cycle).  Both forms give identical results; alt (a schedule choice) swaps them.
template <typename T, int NB, bool STREAM>
static void smooth2d_launch(T *mg, const Level2D &L, int colour, int reps, double omega, hipStream_t s, bool alt)
{
    const long long slots = (long long)L.P.ny * L.P.W;
    const bool split = (NB == 21) != alt;
    if constexpr (NB == 9) {
        if (L.P.tw() > 0) {
            // a tile has at most ceil(tw th / 3) cells of a colour
            const int tw = L.P.tw(), th = L.P.th(), most = kRowAlign - 1 + (tw * th + 2) / 3;
            const dim3 grid((L.ny + th - 1) / th, (most + kTileRows - 1) / kTileRows, (L.nx + tw - 1) / tw);
            if (split)
                hipLaunchKernelGGL((k_smooth2d_split<T, NB, STREAM, true>), grid, dim3(3 * kSplitCells), 0, s, mg, L, colour, omega, reps);
            else
                hipLaunchKernelGGL((k_smooth2d_pass<T, NB, STREAM, true>), grid, dim3(kTileRows), 0, s, mg, L, colour, omega, reps);
            return;
        }
    }
    if (split) {
        dim3 grid((unsigned)((slots + kSplitCells - 1) / kSplitCells));
        hipLaunchKernelGGL((k_smooth2d_split<T, NB, STREAM>), grid, dim3(3 * kSplitCells), 0, s, mg, L, colour, omega, reps);
    } else {
        dim3 grid((unsigned)((slots + 255) / 256));
        hipLaunchKernelGGL((k_smooth2d_pass<T, NB, STREAM>), grid, dim3(256), 0, s, mg, L, colour, omega, reps);
    }
}

hipError_t launch_smooth2d_pass(void *mg, const Level2D &L, int colour, int reps, double omega, int prec,
                               hipStream_t s, int sched)
{
    if (L.P.C != (L.nb == 9 ? 3 : (L.nb == 21 ? 9 : 2))) return hipErrorInvalidValue;
    const bool f32 = prec == NMG_FP32_MG;
    const size_t vsz = f32 ? 4 : 8;
    const bool alt = (sched & (L.nb == 5 ? NMG_SCHED2D_ALT_COARSE : NMG_SCHED2D_ALT_FINEST)) != 0;
    const bool big = !(sched & NMG_SCHED2D_NO_STREAM) && (size_t)L.nb * 9 * (size_t)L.P.M * vsz > kMemCacheBytes;
    // Operators larger than the memory-side cache: on the cross stencil the symmetric schedule
    // returns to colour 1 every other run and to colours 0 and 2 every fourth, so colours 0 and 2
    // stream their rows and leave the cache to colour 1's; with nine colours a colour's rows come
    // back only after the eight others have streamed theirs, so every pass streams.
    const bool stream = big && (L.nb == 21 || (L.nb == 9 && colour != 1));
    if (L.nb == 21) {
        if (f32) { if (stream) smooth2d_launch<float, 21, true>((float *)mg, L, colour, reps, omega, s, alt);
                   else smooth2d_launch<float, 21, false>((float *)mg, L, colour, reps, omega, s, alt); }
        else { if (stream) smooth2d_launch<double, 21, true>((double *)mg, L, colour, reps, omega, s, alt);
               else smooth2d_launch<double, 21, false>((double *)mg, L, colour, reps, omega, s, alt); }
    } else if (L.nb == 9) {
        if (f32) { if (stream) smooth2d_launch<float, 9, true>((float *)mg, L, colour, reps, omega, s, alt);
                   else smooth2d_launch<float, 9, false>((float *)mg, L, colour, reps, omega, s, alt); }
        else { if (stream) smooth2d_launch<double, 9, true>((double *)mg, L, colour, reps, omega, s, alt);
               else smooth2d_launch<double, 9, false>((double *)mg, L, colour, reps, omega, s, alt); }
    } else {
        if (f32) smooth2d_launch<float, 5, false>((float *)mg, L, colour, reps, omega, s, alt);
        else smooth2d_launch<double, 5, false>((double *)mg, L, colour, reps, omega, s, alt);
    }
    return hipGetLastError();
}

// Cells a workgroup of k_resident2d holds: 512 threads have 256 registers each, a row takes 84
// values (nine blocks) or 48 (five points).  Rows are held in FP64, one a thread, or, narrow, two a
// thread: nine-block rows of FP32 levels in FP32 (widened in every pass), five-point rows in FP64.
static int resident2d_cells(int nb, int narrow) { return nb == 21 ? kRes21Cells : (narrow ? 2 * kResNT : kResNT); }

static const void *resident2d_kernel(int nb, int prec, int narrow)
{
    const bool f32 = prec == NMG_FP32_MG;
    if (nb == 21) return f32 ? (const void *)k_resident2d<float, 21, double, 1> : (const void *)k_resident2d<double, 21, double, 1>;
    if (nb == 9 && f32)
        return narrow ? (const void *)k_resident2d<float, 9, float, 2> : (const void *)k_resident2d<float, 9, double, 1>;
    if (nb == 9) return (const void *)k_resident2d<double, 9, double, 1>;
    if (narrow)
        return f32 ? (const void *)k_resident2d<float, 5, double, 2> : (const void *)k_resident2d<double, 5, double, 2>;
    return f32 ? (const void *)k_resident2d<float, 5, double, 1> : (const void *)k_resident2d<double, 5, double, 1>;
}

// The tiling of one resident level: the tile and the passes per exchange with the smallest
// estimated time per pass, out of those whose compute region fits the registers, whose halo fits
// LDS and whose workgroups are all resident at once (one per compute unit).  The estimate: an
// exchange 1.0 us, shared by m passes; a pass `lat` plus `work` per wavefront that a SIMD has to run;
// and a little for every workgroup, so that small levels leave compute units to other streams.  It orders
// the tilings and does not predict times: 64 x 32, FP32, gets 8 x 4 tiles and m = 5 at an estimated
// 0.68 us a pass and takes 1.13.  (A phase may exchange more often than planned: phase2d.)
Resident2D resident2d_plan(const Level2D &L, int prec, int max_wg)
{
    Resident2D best;
    if (L.nb != 21 && L.nb != 9 && L.nb != 5) return best;
    const int C = L.P.C, R = L.nb == 5 ? 1 : 2;
    double cost = 1e30;
    for (int narrow = 0; narrow <= (L.nb == 21 || (L.nb == 9 && prec != NMG_FP32_MG) ? 0 : 1); narrow++) {
        const int cap = resident2d_cells(L.nb, narrow);
        const double lat = 0.2, work = (L.nb == 5 ? 0.16 : 0.28) * (narrow ? 1.5 : 1.0);
        for (int ty = 2; ty <= 32 && ty <= L.ny + 1; ty += 2)
            for (int tx = 4; tx <= 64 && tx <= L.nx + 3; tx += 4) {
                const int gx = (L.nx + tx - 1) / tx, gy = (L.ny + ty - 1) / ty;
                if (gx * gy > max_wg) continue;
                for (int m = 1; m <= 16; m++) {
                    const int hc = R * (m - 1), hd = R * m;
                    const int cw = std::min(tx + 2 * hc, L.nx), ch = std::min(ty + 2 * hc, L.ny);
                    if (cw * ch > cap) break;
                    const int dw = std::min(tx + 2 * hd, L.nx), dh = std::min(ty + 2 * hd, L.ny);
                    const int hw = std::min(2 * hd, L.nx), hh = std::min(2 * hd, L.ny);
                    if (!resident2d_fits(dw, dh)) break;
                    // (a ragged last tile has fewer cells of its own in the same region)
                    if (std::min(dw * dh, tx * hh + ty * hw + hw * hh) > kResHalo * kResNT) break;
                    const double t = (gx * gy > 1 ? 1.0 / m : 0.0) + lat + work * ((cw * ch / C + 255) / 256) + 0.001 * gx * gy;
                    if (t < cost) {
                        cost = t;
                        best.tx = tx; best.ty = ty; best.gx = gx; best.gy = gy; best.m = m; best.narrow = narrow;
                    }
                }
            }
    }
    return best;
}

// workgroups of the kernel that can be resident at once on the current device: one a compute unit
static int cooperative_max_wg(const void *kernel)
{
    int dev = 0, cus = 0, per = 0, coop = 0;
    if (hipGetDevice(&dev) != hipSuccess) return 0;
    if (hipDeviceGetAttribute(&coop, hipDeviceAttributeCooperativeLaunch, dev) != hipSuccess || !coop) return 0;
    if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess) return 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per, kernel, kResNT, 0) != hipSuccess) return 0;
    return per > 0 ? cus : 0;
}

int resident2d_max_wg(int nb, int prec) { return cooperative_max_wg(resident2d_kernel(nb, prec, 0)); }

long long resident2d_max_cells(int nb) { return nb == 21 ? 256LL * kRes21Cells : 1LL << 18; }

size_t resident2d_box_bytes(long long cells, int prec) { return (size_t)2 * cells * 8 * (prec == NMG_FP32_MG ? 3 : 6); }

unsigned resident2d_exchanges(const Level2D &L, int nu, int m) { return (unsigned)((nu * 4LL * (L.P.C - 1) + 1) / m + 2); }

// colour passes of nu smoothing iterations
static int phase_runs(const Level2D &L, int nu) { return nu > 0 ? nu * 4 * (L.P.C - 1) + 1 : 0; }

Resident2D phase2d(const Level2D &L, const Resident2D &G, int nu, int restr)
{
    // fewer passes an exchange than planned only narrow the regions and the halo
    Resident2D H = G;
    if (!restr) H.m = std::max(1, std::min(G.m, phase_runs(L, nu) - 1));
    return H;
}

// every workgroup hears from its neighbours between its first loads and its last stores
static bool phase_exchanges(const Level2D &L, const Resident2D &G, int nu, int restr)
{
    const int runs = phase_runs(L, nu);
    return runs > 0 && (restr || G.m < runs);
}

static Resident2DArgs resident_args(const Level2D &L, const Level2D &Lc, const Resident2D &G, int nu, int prolong, int restr,
                                    unsigned tag, double omega, void *box, long long cells, const NewtonState *state)
{
    Resident2DArgs A;
    A.L = L; A.Lc = Lc;
    A.tx = G.tx; A.ty = G.ty; A.gx = G.gx; A.m = G.m;
    A.nu = nu; A.prolong = prolong; A.restr = restr;
    A.tag = tag; A.omega = omega;
    A.box = (unsigned long long *)box;
    A.cells = cells;
    A.state = state;
    return A;
}

__global__ void k_nothing() {}

hipError_t open_cooperative_queue(hipStream_t s)
{
    return hipLaunchCooperativeKernel(reinterpret_cast<void *>(k_nothing), dim3(1), dim3(64), nullptr, 0, s);
}

hipError_t launch_resident2d(void *mg, const Level2D &L, const Level2D &Lc, const Resident2D &G, int nu, int prolong,
                             int restr, unsigned tag, double omega, void *box, long long cells,
                             const NewtonState *state, int prec, hipStream_t s)
{
    if (G.tx < 2 || L.P.tw() > 0 || L.P.C != (L.nb == 21 ? 9 : (L.nb == 9 ? 3 : 2))) return hipErrorInvalidValue;
    if (!phase_exchanges(L, G, nu, restr)) return hipErrorInvalidValue;
    Resident2DArgs A = resident_args(L, Lc, G, nu, prolong, restr, tag, omega, box, cells, state);
    void *args[] = {&mg, &A};
    return hipLaunchCooperativeKernel(resident2d_kernel(L.nb, prec, G.narrow), dim3(G.gx * G.gy), dim3(kResNT), args, 0, s);
}

Resident2D streamed2d_plan(const Level2D &L, int prec)
{
    Resident2D best;
    if (L.nb != 9 || L.nx % 2 || L.ny % 2 || resident2d_plan(L, prec, 256).tx > 0) return best;
    // the tiling of at most 256 workgroups with the fewest cells a tile; at equal cells the squarest, whose halo is smallest
    long long cost = 1LL << 60;
    for (int ty = 4; ty <= 64 && ty <= L.ny + 1; ty += 2)
        for (int tx = 16; tx <= 96 && tx <= L.nx + 1; tx += 2) {
            const int gx = (L.nx + tx - 1) / tx, gy = (L.ny + ty - 1) / ty;
            if (gx * gy > 256 || (tx + 4) * (ty + 4) > kStrCells || 4 * (tx + ty) > kResNT) continue;
            const long long t = (long long)tx * ty * 1024 + 4 * (tx + ty);
            if (t < cost) {
                cost = t;
                best.tx = tx; best.ty = ty; best.gx = gx; best.gy = gy; best.m = 1;
            }
        }
    return best;
}

static const void *streamed2d_kernel(int prec)
{
    return prec == NMG_FP32_MG ? (const void *)k_streamed2d<float, 2> : (const void *)k_streamed2d<double, 1>;
}

int streamed2d_max_wg(int prec) { return cooperative_max_wg(streamed2d_kernel(prec)); }

hipError_t launch_streamed2d(void *mg, const Level2D &L, const Level2D &Lc, const Resident2D &G, int nu, int prolong,
                             int restr, unsigned tag, double omega, void *box, long long cells,
                             const NewtonState *state, int prec, hipStream_t s)
{
    if (G.tx < 2 || L.P.tw() != G.tx || L.P.th() != G.ty || L.P.nx() != L.nx) return hipErrorInvalidValue;
    if (!phase_exchanges(L, G, nu, restr)) return hipErrorInvalidValue;
    Resident2DArgs A = resident_args(L, Lc, G, nu, prolong, restr, tag, omega, box, cells, state);
    void *args[] = {&mg, &A};
    return hipLaunchCooperativeKernel(streamed2d_kernel(prec), dim3(G.gx * G.gy), dim3(kResNT), args, 0, s);
}

hipError_t launch_restrict2d(void *mg, const Level2D &Lf, const Level2D &Lc, int prec, hipStream_t s)
{
    dim3 grid((Lf.nx + kRX - 1) / kRX, Lc.ny);
    DISPATCH(prec, k_restrict2d, grid, dim3(2 * kRX), Lf, Lc);
    return hipGetLastError();
}

hipError_t launch_prolong2d(void *mg, const Level2D &Lf, const Level2D &Lc, int prec, hipStream_t s)
{
    dim3 grid((Lf.nx + 63) / 64, (Lf.ny + 3) / 4);
    DISPATCH(prec, k_prolong2d, grid, dim3(64, 4), Lf, Lc);
    return hipGetLastError();
}

hipError_t launch_coarse_factor2d(void *mg, const Level2D &L, double *lu, int prec, hipStream_t s)
{
    DISPATCH(prec, k_coarse_factor2d, dim3(1), dim3(1024), L, lu);
    return hipGetLastError();
}

hipError_t launch_sweeps2d(void *mg, const Level2D &L, int nu, double omega, int prec, hipStream_t s)
{
    const bool f32 = prec == NMG_FP32_MG;
    if (L.nb == 21) {
        if (f32) hipLaunchKernelGGL((k_sweeps2d<float, 21>), dim3(1), dim3(1024), 0, s, (float *)mg, L, nu, omega);
        else hipLaunchKernelGGL((k_sweeps2d<double, 21>), dim3(1), dim3(1024), 0, s, (double *)mg, L, nu, omega);
    } else if (L.nb == 9) {
        if (f32) hipLaunchKernelGGL((k_sweeps2d<float, 9>), dim3(1), dim3(1024), 0, s, (float *)mg, L, nu, omega);
        else hipLaunchKernelGGL((k_sweeps2d<double, 9>), dim3(1), dim3(1024), 0, s, (double *)mg, L, nu, omega);
    } else {
        if (f32) hipLaunchKernelGGL((k_sweeps2d<float, 5>), dim3(1), dim3(1024), 0, s, (float *)mg, L, nu, omega);
        else hipLaunchKernelGGL((k_sweeps2d<double, 5>), dim3(1), dim3(1024), 0, s, (double *)mg, L, nu, omega);
    }
    return hipGetLastError();
}

hipError_t launch_bottom2d(void *mg, const Level2D *levels, int first, int nlev, int nu1, int nu2, double omega,
                           const double *lu, int prec, hipStream_t s, int sweeps)
{
    if (first < 0 || first >= nlev || nlev > kMaxLevels) return hipErrorInvalidValue;
    Bottom2DArgs B;
    memset(&B, 0, sizeof(B));
    for (int l = 0; l < nlev; l++) B.L[l] = levels[l];
    B.first = first;
    B.levels = nlev;
    B.nu1 = nu1;
    B.nu2 = nu2;
    B.omega = omega;
    B.lu = lu;
    B.sweeps = sweeps;
    const int nbf = levels[first].nb;
    const bool f32 = prec == NMG_FP32_MG;
    float *mf = (float *)mg;
    double *md = (double *)mg;
    if (nbf == 21) {
        if (f32) hipLaunchKernelGGL((k_bottom2d<float, 21>), dim3(1), dim3(512), 0, s, mf, B);
        else hipLaunchKernelGGL((k_bottom2d<double, 21>), dim3(1), dim3(512), 0, s, md, B);
    } else if (nbf == 9) {
        if (f32) hipLaunchKernelGGL((k_bottom2d<float, 9>), dim3(1), dim3(512), 0, s, mf, B);
        else hipLaunchKernelGGL((k_bottom2d<double, 9>), dim3(1), dim3(512), 0, s, md, B);
    } else {
        if (f32) hipLaunchKernelGGL((k_bottom2d<float, 5>), dim3(1), dim3(512), 0, s, mf, B);
        else hipLaunchKernelGGL((k_bottom2d<double, 5>), dim3(1), dim3(512), 0, s, md, B);
    }
    return hipGetLastError();
}

hipError_t launch_fill(void *p, int prec, long long n, hipStream_t s)
{
    int blocks = (int)std::min<long long>((n + 255) / 256, 4096);
    if (blocks < 1) return hipSuccess;
    if (prec == NMG_FP32_MG) hipLaunchKernelGGL(k_fill<float>, dim3(blocks), dim3(256), 0, s, (float *)p, n);
    else hipLaunchKernelGGL(k_fill<double>, dim3(blocks), dim3(256), 0, s, (double *)p, n);
    return hipGetLastError();
}

hipError_t launch_update2d(double *U, const void *mg, const Level2D &L0, double tau, const NewtonState *state,
                           int prec, hipStream_t s)
{
    const long long n = 3LL * L0.nx * L0.ny;
    int blocks = (int)std::min<long long>((n + 255) / 256, 8192);
    if (prec == NMG_FP32_MG)
        hipLaunchKernelGGL(k_update2d<float>, dim3(blocks), dim3(256), 0, s, U, (const float *)mg, L0, tau, state);
    else
        hipLaunchKernelGGL(k_update2d<double>, dim3(blocks), dim3(256), 0, s, U, (const double *)mg, L0, tau, state);
    return hipGetLastError();
}

hipError_t launch_dinv2d(const double *J, void *Dinv, const Level2D &L0, int prec, hipStream_t s)
{
    const long long n = (long long)L0.nx * L0.ny;
    int blocks = (int)std::min<long long>((n + 255) / 256, 8192);
    if (prec == NMG_FP32_MG) hipLaunchKernelGGL(k_dinv2d<float>, dim3(blocks), dim3(256), 0, s, J, (float *)Dinv, L0);
    else hipLaunchKernelGGL(k_dinv2d<double>, dim3(blocks), dim3(256), 0, s, J, (double *)Dinv, L0);
    return hipGetLastError();
}

hipError_t launch_permute2d(const void *src, int src_prec, void *dst, int dst_prec, const Level2D &L, int nent,
                            int rows, int to_level, hipStream_t s)
{
    const long long total = (long long)L.nx * L.ny * nent;
    int blocks = (int)std::min<long long>((total + 255) / 256, 16384);
    if (blocks < 1) return hipSuccess;
    const bool s32 = src_prec == NMG_FP32_MG, d32 = dst_prec == NMG_FP32_MG;
    if (!s32 && !d32)
        hipLaunchKernelGGL((k_permute2d<double, double>), dim3(blocks), dim3(256), 0, s, (const double *)src,
                           (double *)dst, L, nent, rows, to_level);
    else if (!s32)
        hipLaunchKernelGGL((k_permute2d<double, float>), dim3(blocks), dim3(256), 0, s, (const double *)src,
                           (float *)dst, L, nent, rows, to_level);
    else if (!d32)
        hipLaunchKernelGGL((k_permute2d<float, double>), dim3(blocks), dim3(256), 0, s, (const float *)src,
                           (double *)dst, L, nent, rows, to_level);
    else
        hipLaunchKernelGGL((k_permute2d<float, float>), dim3(blocks), dim3(256), 0, s, (const float *)src,
                           (float *)dst, L, nent, rows, to_level);
    return hipGetLastError();
}

hipError_t launch_state2d(const double *partial, int ntiles, long long ncells, double tol, int n_max,
                          NewtonState *state, double *hist, int max_hist, int init, hipStream_t s)
{
    hipLaunchKernelGGL(k_state2d, dim3(1), dim3(256), 0, s, partial, ntiles, ncells, tol, n_max, state, hist,
                       max_hist, init);
    return hipGetLastError();
}

}  // namespace nmg
