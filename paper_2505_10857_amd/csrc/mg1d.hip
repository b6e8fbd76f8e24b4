// Geometric multigrid for the 1D regularised Newton systems (section 3.4, eq. 15-19,
// Algorithm 2) on gfx950.
//
//  * k_coarsen: coarse operators of eq. (17) for up to ten levels in one launch.  A workgroup
//    owns an aligned run of 1024 cells of the starting level and reduces them level by level
//    in LDS (each coarse cell aggregates two children, eq. 15), writing every level's blocks.
//    The smoothers form the closed-form 2x2 inverses of the diagonal blocks of eq. (19)
//    themselves, so no inverse is stored.
//  * k_smooth: all nu multicolour block-SOR half-sweeps of one smoothing phase fused in one
//    launch.  Each workgroup loads its cells' block rows and right-hand side into
//    registers once, keeps dU in LDS, and runs the half-sweeps with a halo wide enough that
//    the cells it writes are exact; the pre-smoothing kernel then forms the restricted
//    right-hand side of eq. (17), the post-smoothing kernel first adds the prolongation of
//    eq. (18) (and, at the finest level after the last cycle, applies the Newton update of
//    eq. 14).  HBM traffic per level and phase is one read of the operator.
//  * k_group: the same for up to four levels of a tile in one launch, for few cells in all.
//  * k_bottom: all small levels of one instance in one workgroup: smoothing and restriction
//    down, the coarsest system solved exactly (up to rounding) by block parallel cyclic
//    reduction, prolongation and smoothing back up.
// The last two hold a level as pairs of cells with one parent (PairLevel), neighbours in adjacent
// lanes.
#include "nmg_common.h"

namespace nmg {

template <typename T>
__device__ __forceinline__ double ld(const T *p, long long i) { return (double)p[i]; }

__device__ __forceinline__ bool active_of(const MGArgs &mg, int inst)
{
    return mg.state == nullptr || mg.state[mg.insts[inst].active_idx].active;
}

// The inverse of a 2x2 block.  The four quotients share the divisor's reciprocal where that is far
// from overflow and denormals: refined by two Newton-Raphson steps, each quotient corrected once by
// its residual (Markstein), which rounds as the division does.
__device__ __forceinline__ void inv2(const double A[4], double B[4])
{
    double det = A[0] * A[3] - A[1] * A[2];
    if (fabs(det) > 0x1p-400 && fabs(det) < 0x1p400) {
        double r = __builtin_amdgcn_rcp(det);
        r = fma(fma(-det, r, 1.0), r, r);
        r = fma(fma(-det, r, 1.0), r, r);
        const double N[4] = {A[3], -A[1], -A[2], A[0]};
#pragma unroll
        for (int e = 0; e < 4; e++) {
            const double q = N[e] * r;
            B[e] = fma(fma(-det, q, N[e]), r, q);
        }
        return;
    }
    B[0] = A[3] / det;
    B[1] = -A[1] / det;
    B[2] = -A[2] / det;
    B[3] = A[0] / det;
}

// ---- coarse operators --------------------------------------------------------------------

// Children blocks (b = 0..nb-1 <-> column offsets -nb/2..nb/2) of cells 2jc and 2jc+1 ->
// coarse tridiagonal row of cell jc, summing the fine blocks of eq. (17) in order of the
// child row and then the child column.
__device__ __forceinline__ void coarse_row(int nb, const double (*f0)[4], const double (*f1)[4],
                                           double Wc[4], double Dc[4], double Ec[4])
{
#pragma unroll
    for (int e = 0; e < 4; e++) {
        if (nb == 5) {
            Wc[e] = f0[0][e] + f0[1][e] + f1[0][e];
            Dc[e] = f0[2][e] + f0[3][e] + f1[1][e] + f1[2][e];
            Ec[e] = f0[4][e] + f1[3][e] + f1[4][e];
        } else {
            Wc[e] = f0[0][e];
            Dc[e] = f0[1][e] + f0[2][e] + f1[0][e] + f1[1][e];
            Ec[e] = f1[2][e];
        }
    }
}

template <typename T, int NB>
__device__ __forceinline__ void first_coarse(const Level1D &L0, const Level1D &Lc, T *base, int c0,
                                             int t, double (*blk)[12])
{
    for (int k = 0; k < kCoarsenCells / 2; k++) {
        const int jl = t * (kCoarsenCells / 2) + k;   // local coarse index
        const int jc = c0 + jl;
        if (jc >= Lc.n) break;
        double f0[5][4], f1[5][4];
#pragma unroll
        for (int b = 0; b < NB; b++)
#pragma unroll
            for (int e = 0; e < 4; e++) {
                f0[b][e] = ld(base + L0.J, (b * 4 + e) * (long long)L0.n + 2 * jc);
                f1[b][e] = ld(base + L0.J, (b * 4 + e) * (long long)L0.n + 2 * jc + 1);
            }
        double W[4], D[4], E[4];
        coarse_row(NB, f0, f1, W, D, E);
#pragma unroll
        for (int e = 0; e < 4; e++) {
            blk[jl][e] = W[e]; blk[jl][4 + e] = D[e]; blk[jl][8 + e] = E[e];
            base[Lc.J + (0 * 4 + e) * (long long)Lc.n + jc] = (T)W[e];
            base[Lc.J + (1 * 4 + e) * (long long)Lc.n + jc] = (T)D[e];
            base[Lc.J + (2 * 4 + e) * (long long)Lc.n + jc] = (T)E[e];
        }
    }
}

template <typename T>
__global__ void __launch_bounds__(kTile) k_coarsen(MGArgs mg, const Tile *tiles)
{
    constexpr int CPT = kCoarsenCells;           // level-l0 cells per thread
    constexpr int SPAN = kTile * CPT;             // level-l0 cells per workgroup
    __shared__ double blk[SPAN / 2][12];          // current coarse level: W, D, E per cell
    const Tile tl = tiles[blockIdx.x];
    const Level1D L0 = mg.levs[tl.lev];
    if (!active_of(mg, L0.inst)) return;
    T *base = reinterpret_cast<T *>(mg.mg);
    const int t = threadIdx.x;
    const int nb = L0.nb;

    if (L0.coarsest) return;

    // first coarse level from the starting level (global reads)
    int lev = L0.child;
    Level1D Lc = mg.levs[lev];
    const int c0 = tl.a / 2;                      // first coarse cell of this tile
    if (nb == 5) first_coarse<T, 5>(L0, Lc, base, c0, t, blk);
    else first_coarse<T, 3>(L0, Lc, base, c0, t, blk);
    __syncthreads();

    // further levels from LDS
    int cnt = SPAN / 2;     // cells of the current level held by this tile
    int cstart = c0;        // first cell (level index) of the current level in this tile
    while (!Lc.coarsest && cnt >= 2) {
        const int nlev = Lc.child;
        const Level1D Ln = mg.levs[nlev];
        const int nstart = cstart / 2;
        const int ncnt = cnt / 2;
        double W[4], D[4], E[4];
        const int jc = nstart + t;
        const bool mine = t < ncnt && jc < Ln.n;
        if (mine) {
            double f0[5][4], f1[5][4];
#pragma unroll
            for (int e = 0; e < 4; e++) {
                f0[0][e] = blk[2 * t][e]; f0[1][e] = blk[2 * t][4 + e]; f0[2][e] = blk[2 * t][8 + e];
                f1[0][e] = blk[2 * t + 1][e]; f1[1][e] = blk[2 * t + 1][4 + e]; f1[2][e] = blk[2 * t + 1][8 + e];
            }
            coarse_row(3, f0, f1, W, D, E);
        }
        __syncthreads();
        if (mine) {
            for (int e = 0; e < 4; e++) {
                blk[t][e] = W[e]; blk[t][4 + e] = D[e]; blk[t][8 + e] = E[e];
                base[Ln.J + (0 * 4 + e) * (long long)Ln.n + jc] = (T)W[e];
                base[Ln.J + (1 * 4 + e) * (long long)Ln.n + jc] = (T)D[e];
                base[Ln.J + (2 * 4 + e) * (long long)Ln.n + jc] = (T)E[e];
            }
        }
        __syncthreads();
        Lc = Ln;
        cnt = ncnt;
        cstart = nstart;
    }
}

// ---- fused smoother ------------------------------------------------------------------------

// mode 0: (zero or loaded) dU -> nu1 symmetric steps -> write dU, restrict rhs to the child.
// mode 1: dU + prolongated child dU -> nu2 symmetric steps -> write dU (or update U).
// mode 2: dU + prolongated child dU -> nu2 + nu1 symmetric steps (the post-smoothing of one
//         V-cycle and the pre-smoothing of the next, with nothing between them on this level)
//         -> write dU, restrict rhs to the child; its tiles have the wider halo halo2.
// src_out: the tile reads dU from dUo (1) or dU (0) and writes its cells to the other buffer.
template <typename T, int NB, int MODE, int TW>
__global__ void __launch_bounds__(TW) k_smooth(MGArgs mg, const Tile *tiles, int zero_init,
                                                  int final_update, int src_out, int reverse)
{
    constexpr int mode = MODE;
    constexpr int HW = NB / 2;
    constexpr int C = NB == 5 ? 3 : 2;
    __shared__ double s0[TW + 2 * HW], s1[TW + 2 * HW];
    // reverse: the last tiles first (workgroups start roughly in index order), so that a pass
    // that follows another pass over the same data begins with what that pass touched last,
    // which is still in the memory-side cache
    const Tile tl = tiles[reverse ? gridDim.x - 1 - blockIdx.x : blockIdx.x];
    const Level1D L = mg.levs[tl.lev];
    if (L.nb != NB) return;
    if (!active_of(mg, L.inst)) return;
    const Inst1D &I = mg.insts[L.inst];
    T *base = reinterpret_cast<T *>(mg.mg);
    const int n = L.n, h = mode == 2 ? L.halo2 : L.halo, V = mode == 2 ? L.V2 : L.V;
    const int t = threadIdx.x;
    const int j = tl.a - h + t;
    const bool in = j >= 0 && j < n;
    // the halo of a tile must hold the values from before the launch, so the cells are written
    // to the other buffer
    const long long src = src_out ? L.dUo : L.dU, dst = src_out ? L.dU : L.dUo;

    double Jr[NB][4], D[4], r0 = 0.0, r1 = 0.0, du0 = 0.0, du1 = 0.0;
#pragma unroll
    for (int b = 0; b < NB; b++)
#pragma unroll
        for (int e = 0; e < 4; e++) Jr[b][e] = in ? ld(base + L.J, (b * 4 + e) * (long long)n + j) : 0.0;
    // the inverse of the diagonal block, formed here instead of read (one division per cell
    // and launch against 4 values of HBM traffic per cell and half-sweep phase)
    if (in) inv2(Jr[HW], D);
    else D[0] = D[1] = D[2] = D[3] = 0.0;
    if (in) {
        r0 = ld(base + L.rhs, j);
        r1 = ld(base + L.rhs, n + (long long)j);
        if (!(mode == 0 && zero_init)) {
            du0 = ld(base + src, j);
            du1 = ld(base + src, n + (long long)j);
        }
        if (mode != 0) {
            const Level1D &Lc = mg.levs[L.child];
            du0 = du0 + ld(base + Lc.dU, j >> 1);
            du1 = du1 + ld(base + Lc.dU, Lc.n + (long long)(j >> 1));
        }
    }
    s0[t + HW] = du0;
    s1[t + HW] = du1;
    if (t < HW) { s0[t] = 0.0; s1[t] = 0.0; s0[TW + HW + t] = 0.0; s1[TW + HW + t] = 0.0; }
    __syncthreads();

    const double w = I.omega;
    const int col = ((j % C) + C) % C;
    // mode 2 runs the post-smoothing steps, rounds dU to the storage type as the separate
    // launches would when storing it, then the pre-smoothing steps
    for (int phase = 0; phase < (mode == 2 ? 2 : 1); phase++) {
        const int steps = mode == 0 ? I.nu1 : mode == 1 ? I.nu2 : phase == 0 ? I.nu2 : I.nu1;
        if (phase == 1) {
            du0 = (double)(T)du0;
            du1 = (double)(T)du1;
            s0[t + HW] = du0;
            s1[t + HW] = du1;
            __syncthreads();
        }
        // half-sweep colours 0..C-1, C-1..0 per step; a run of equal colours (at every turn)
        // sees the same neighbour values, so its relaxations share one off-diagonal sum
        const int total = steps * 2 * C;
        int cur = -1, reps = 0;
        for (int q = 0; q <= total; q++) {
            const int hs = q % (2 * C);
            const int c = q == total ? -1 : (hs < C ? hs : 2 * C - 1 - hs);
            if (c == cur) { reps++; continue; }
            if (reps > 0) {
                if (in && col == cur) {
                    // eq. (19): dU_j <- (1-w) dU_j - w J_jj^{-1} (rhs_j + sum_{i != j} J_ji dU_i)
                    double a0 = r0, a1 = r1;
#pragma unroll
                    for (int b = 0; b < NB; b++) {
                        if (b == HW) continue;
                        const double x0 = s0[t + b], x1 = s1[t + b];
                        a0 = a0 + (Jr[b][0] * x0 + Jr[b][1] * x1);
                        a1 = a1 + (Jr[b][2] * x0 + Jr[b][3] * x1);
                    }
                    const double t0 = D[0] * a0 + D[1] * a1;
                    const double t1 = D[2] * a0 + D[3] * a1;
                    for (int k = 0; k < reps; k++) {
                        du0 = (1.0 - w) * du0 - w * t0;
                        du1 = (1.0 - w) * du1 - w * t1;
                    }
                    s0[t + HW] = du0;
                    s1[t + HW] = du1;
                }
                __syncthreads();
            }
            cur = c;
            reps = 1;
        }
    }

    const bool valid = in && t >= h && t < h + V;
    if (mode != 1) {
        // restriction, eq. (17): rhs_c = sum over the two children of (rhs + sum_i J dU_i)
        double a0 = r0, a1 = r1;
#pragma unroll
        for (int b = 0; b < NB; b++) {
            const double x0 = s0[t + b], x1 = s1[t + b];
            a0 = a0 + (Jr[b][0] * x0 + Jr[b][1] * x1);
            a1 = a1 + (Jr[b][2] * x0 + Jr[b][3] * x1);
        }
        const double p0 = __shfl_xor(a0, 1, 64);
        const double p1 = __shfl_xor(a1, 1, 64);
        if (valid) {
            base[dst + j] = (T)du0;
            base[dst + n + (long long)j] = (T)du1;
            if ((j & 1) == 0 && !L.coarsest) {
                const Level1D &Lc = mg.levs[L.child];
                base[Lc.rhs + (j >> 1)] = (T)(a0 + p0);
                base[Lc.rhs + Lc.n + (long long)(j >> 1)] = (T)(a1 + p1);
            }
        }
    } else if (valid) {
        if (final_update) {
            // eq. (14): U <- U + tau dU
            I.U[j] = I.U[j] + I.tau * du0;
            I.U[I.N + j] = I.U[I.N + j] + I.tau * du1;
        } else {
            base[dst + j] = (T)du0;
            base[dst + n + (long long)j] = (T)du1;
        }
    }
}

// ---- coarsest level ------------------------------------------------------------------------
// The coarsest system  W_j x_{j-1} + D_j x_j + E_j x_{j+1} = -rhs_j  (2x2 blocks) is solved
// exactly by block parallel cyclic reduction: step k (stride s = 2^k) eliminates the couplings
// at distance s from every row at once,
//     a_j = -W_j D_{j-s}^{-1},  g_j = -E_j D_{j+s}^{-1},
//     W_j <- a_j W_{j-s},  E_j <- g_j E_{j+s},  D_j <- D_j + a_j E_{j-s} + g_j W_{j+s},
// and the same combination of right-hand sides; after ceil(log2 n) steps every row is
// decoupled and x_j = D_j^{-1} b_j.  One thread per cell, 2x2 blocks in LDS, inside the
// bottom-of-cycle kernel below.

__device__ __forceinline__ void mul2(const double A[4], const double B[4], double C[4])
{
    C[0] = A[0] * B[0] + A[1] * B[2];
    C[1] = A[0] * B[1] + A[1] * B[3];
    C[2] = A[2] * B[0] + A[3] * B[2];
    C[3] = A[2] * B[1] + A[3] * B[3];
}

// ---- bottom of the V-cycle -----------------------------------------------------------------
// Every level with at most 2 K NT cells (always including the coarsest; the plan picks the first
// such level) is handled by one NT-thread workgroup per instance in a single launch:
// pre-smoothing and restriction down to the coarsest level, the cyclic-reduction solve there,
// prolongation and post-smoothing back up.
//
// A thread owns the two children 2p and 2p + 1 of one coarse cell (K such pairs on the first
// level): every lane has a cell to relax in each half-sweep, one neighbour of each cell is the
// thread's own, the restriction adds the thread's own two sums and the prolongation reads one
// parent.  A level's rows are read as pairs while the level before it is being smoothed, so the
// chain of levels waits for memory once; the rhs and the pre-smoothed dU of all levels but the
// first stay in LDS, rounded to the storage type.  What is left is the chain itself: about 400
// cycles a half-sweep (a barrier, one LDS round trip and the dependent FP64 operations of a
// cell), 2 nu + 1 of them a level each way, and 500 a reduction step.
// Same arithmetic, in the same order, as the per-level kernels.

constexpr int kBottomNT = 512;

// vectors of two neighbouring cells, readable at the alignment of one value
template <typename T> struct Two;
template <> struct Two<double> { typedef double v __attribute__((ext_vector_type(2), aligned(8))); };
template <> struct Two<float> { typedef float v __attribute__((ext_vector_type(2), aligned(4))); };

template <typename T> __device__ __forceinline__ typename Two<T>::v ld2(const T *p)
{
    return *reinterpret_cast<const typename Two<T>::v *>(p);
}
template <typename T> __device__ __forceinline__ void st2(T *p, T a, T b)
{
    typename Two<T>::v x;
    x.x = a;
    x.y = b;
    *reinterpret_cast<typename Two<T>::v *>(p) = x;
}

template <typename T> struct PairRows { typename Two<T>::v j[12]; };   // W, D, E of two cells

struct Vec2d { double a, b; };             // the two components of one cell in LDS

template <typename T>
__device__ __forceinline__ void load_rows(PairRows<T> &R, const T *J, int n, int p)
{
#pragma unroll
    for (int e = 0; e < 12; e++) R.j[e] = ld2(J + e * (long long)n + 2 * p);
}

// the value of the lane before (0 in lane 0) or after (0 in lane 63), DPP wave_shr:1 / wave_shl:1
template <int CTRL>
__device__ __forceinline__ double lane_shift(double x)
{
    const unsigned long long v = __double_as_longlong(x);
    const int lo = __builtin_amdgcn_update_dpp(0, (int)(unsigned)v, CTRL, 0xf, 0xf, true);
    const int hi = __builtin_amdgcn_update_dpp(0, (int)(v >> 32), CTRL, 0xf, 0xf, true);
    return __longlong_as_double(((long long)hi << 32) | (unsigned)lo);
}
__device__ __forceinline__ Vec2d lane_before(double a, double b) { return Vec2d{lane_shift<0x138>(a), lane_shift<0x138>(b)}; }
__device__ __forceinline__ Vec2d lane_after(double a, double b) { return Vec2d{lane_shift<0x130>(a), lane_shift<0x130>(b)}; }

__device__ __forceinline__ double of_lane(double x, int lane)
{
    const unsigned long long v = __double_as_longlong(x);
    const int lo = __builtin_amdgcn_readlane((int)(unsigned)v, lane), hi = __builtin_amdgcn_readlane((int)(v >> 32), lane);
    return __longlong_as_double(((long long)hi << 32) | (unsigned)lo);
}

// Where a level's np pairs lie: wavefront v holds the 64 K pairs from p0 on, and its own ones, whose
// results are used, are the first to last of them.  Windows: neighbouring wavefronts overlap by g
// pairs each way, as far as wrong values travel from a window's edge in the steps of one level, so
// that no half-sweep waits for another wavefront (620 cycles one with a barrier and the edge cells
// through LDS, 320 so).  A level too large for windows is split without overlap.
struct PairPlace {
    int p0, lo, hi, first, last, lane, wave, nw;
    bool sync;

    // np pairs on nwaves wavefronts from w0 on; those from lo to hi - 1 exist
    __device__ __forceinline__ PairPlace(int np, int lo_, int hi_, int K, int g, int t, int w0, int nwaves) : lo(lo_), hi(hi_)
    {
        lane = t & 63;
        wave = __builtin_amdgcn_readfirstlane(t >> 6) - w0;
        const int own = 64 * K - 2 * g;
        const bool window = np > 64 * K && own > 0 && np <= own * nwaves;
        const int stride = window ? own : 64 * K;
        nw = window ? nwaves : (np + 64 * K - 1) / (64 * K);
        first = window ? g : 0;
        last = first + stride;
        p0 = wave * stride - first;
        sync = nw > 1 && !window;
    }
    __device__ __forceinline__ int pair(int k) const { return p0 + 64 * k + lane; }
    __device__ __forceinline__ bool on() const { return wave >= 0 && wave < nw; }
    // the pair exists / is this wavefront's to write
    __device__ __forceinline__ bool in(int k) const { return on() && pair(k) >= lo && pair(k) < hi; }
    __device__ __forceinline__ bool own(int k) const
    {
        return in(k) && 64 * k + lane >= first && 64 * k + lane < last;
    }
};

// Pairs of a level in registers: r and du are (cell 2p: 0, 1; cell 2p + 1: 2, 3), zero where there
// is no pair.  Neighbours come from the adjacent lanes; without windows, what crosses two wavefronts
// goes through LDS: sl[v] is the last cell before wavefront v's, sr[v] the first cell of wavefront v.
template <typename T, int K>
struct PairLevel {
    double D[K][2][4], r[K][4], du[K][4];

    __device__ __forceinline__ void inverses(const PairRows<T> (&R)[K], const PairPlace &P)
    {
#pragma unroll
        for (int k = 0; k < K; k++) {
            if (!P.in(k)) continue;
            const double A0[4] = {(double)R[k].j[4].x, (double)R[k].j[5].x, (double)R[k].j[6].x, (double)R[k].j[7].x};
            const double A1[4] = {(double)R[k].j[4].y, (double)R[k].j[5].y, (double)R[k].j[6].y, (double)R[k].j[7].y};
            inv2(A0, D[k][0]);
            inv2(A1, D[k][1]);
        }
    }

    // a + W x (+ D c) + E y of one cell of a pair
    template <int S, bool DIAG>
    static __device__ __forceinline__ void row(const PairRows<T> &R, Vec2d x, Vec2d c, Vec2d y, double &a0, double &a1)
    {
        auto J = [&](int e) { return (double)(S ? R.j[e].y : R.j[e].x); };
        a0 = a0 + (J(0) * x.a + J(1) * x.b);
        a1 = a1 + (J(2) * x.a + J(3) * x.b);
        if (DIAG) {
            a0 = a0 + (J(4) * c.a + J(5) * c.b);
            a1 = a1 + (J(6) * c.a + J(7) * c.b);
        }
        a0 = a0 + (J(8) * y.a + J(9) * y.b);
        a1 = a1 + (J(10) * y.a + J(11) * y.b);
    }

    template <int S>
    __device__ __forceinline__ void relax(int k, const PairRows<T> &R, Vec2d x, Vec2d y, double w, bool twice)
    {
        double a0 = r[k][2 * S], a1 = r[k][2 * S + 1];
        row<S, false>(R, x, x, y, a0, a1);
        const double t0 = D[k][S][0] * a0 + D[k][S][1] * a1;
        const double t1 = D[k][S][2] * a0 + D[k][S][3] * a1;
        const double v = 1.0 - w, s0 = w * t0, s1 = w * t1;
        du[k][2 * S] = v * du[k][2 * S] - s0;
        du[k][2 * S + 1] = v * du[k][2 * S + 1] - s1;
        if (twice) {
            du[k][2 * S] = v * du[k][2 * S] - s0;
            du[k][2 * S + 1] = v * du[k][2 * S + 1] - s1;
        }
    }

    // the odd cell before pair(k), the even cell after it
    __device__ __forceinline__ Vec2d before(int k, Vec2d edge, int lane) const
    {
        Vec2d x = lane_before(du[k][2], du[k][3]);
        const Vec2d e = k > 0 ? Vec2d{of_lane(du[k > 0 ? k - 1 : 0][2], 63), of_lane(du[k > 0 ? k - 1 : 0][3], 63)} : edge;
        return lane == 0 ? e : x;
    }
    __device__ __forceinline__ Vec2d after(int k, Vec2d edge, int lane) const
    {
        Vec2d y = lane_after(du[k][0], du[k][1]);
        const Vec2d e = k < K - 1 ? Vec2d{of_lane(du[k < K - 1 ? k + 1 : 0][0], 0), of_lane(du[k < K - 1 ? k + 1 : 0][1], 0)} : edge;
        return lane == 63 ? e : y;
    }

    template <bool SYNC, bool TWICE>
    __device__ __forceinline__ void even(const PairRows<T> (&R)[K], const PairPlace &P, double w, const Vec2d *sl, Vec2d *sr)
    {
        if (!SYNC || P.on()) {
            Vec2d edge = Vec2d{0.0, 0.0};
            if (SYNC) edge = sl[P.wave];
            Vec2d x[K];
#pragma unroll
            for (int k = 0; k < K; k++) x[k] = before(k, edge, P.lane);
#pragma unroll
            for (int k = K - 1; k >= 0; k--)
                if (P.in(k)) relax<0>(k, R[k], x[k], Vec2d{du[k][2], du[k][3]}, w, TWICE);
            if (SYNC && P.lane == 0) sr[P.wave] = Vec2d{du[0][0], du[0][1]};
        }
        if (SYNC) __syncthreads();
    }
    template <bool SYNC>
    __device__ __forceinline__ void odd(const PairRows<T> (&R)[K], const PairPlace &P, double w, Vec2d *sl, const Vec2d *sr)
    {
        if (!SYNC || P.on()) {
            Vec2d edge = Vec2d{0.0, 0.0};
            if (SYNC) edge = sr[P.wave + 1];
            Vec2d y[K];
#pragma unroll
            for (int k = 0; k < K; k++) y[k] = after(k, edge, P.lane);
#pragma unroll
            for (int k = 0; k < K; k++)
                if (P.in(k)) relax<1>(k, R[k], Vec2d{du[k][0], du[k][1]}, y[k], w, true);
            if (SYNC && P.lane == 63) sl[P.wave + 1] = Vec2d{du[K - 1][2], du[K - 1][3]};
        }
        if (SYNC) __syncthreads();
    }

    // nu symmetric steps from the dU in the registers.  Half-sweeps 0 1 1 0 per step: runs 0,
    // (1 1), (0 0), ..., (1 1), 0 of one colour share the neighbour values and so one
    // off-diagonal sum.
    template <bool SYNC>
    __device__ __forceinline__ void sweeps(int nu, double w, const PairRows<T> (&R)[K], const PairPlace &P, Vec2d *sl, Vec2d *sr)
    {
        if (nu <= 0) return;
        even<SYNC, false>(R, P, w, sl, sr);
        for (int i = 1; i < nu; i++) {
            odd<SYNC>(R, P, w, sl, sr);
            even<SYNC, true>(R, P, w, sl, sr);
        }
        odd<SYNC>(R, P, w, sl, sr);
        even<SYNC, false>(R, P, w, sl, sr);
    }
    __device__ __forceinline__ void smooth(int nu, double w, const PairRows<T> (&R)[K], const PairPlace &P, Vec2d *sl, Vec2d *sr)
    {
        if (!P.sync) {
            if (P.on()) sweeps<false>(nu, w, R, P, sl, sr);
            return;
        }
        if (P.on()) {
            if (P.lane == 63) sl[P.wave + 1] = Vec2d{du[K - 1][2], du[K - 1][3]};
            if (P.lane == 0) {
                sr[P.wave] = Vec2d{du[0][0], du[0][1]};
                if (P.wave == 0) sl[0] = Vec2d{0.0, 0.0};
                if (P.wave == P.nw - 1) sr[P.nw] = Vec2d{0.0, 0.0};
            }
        }
        __syncthreads();
        sweeps<true>(nu, w, R, P, sl, sr);
    }

    // restriction to the child (eq. 17): rhs + J dU summed over the pair, rounded to the value
    // type as the tiled kernels round it in HBM, so the result does not depend on which levels
    // run here
    __device__ __forceinline__ void restrict_to(T *q0, T *q1, const PairRows<T> (&R)[K], const PairPlace &P, const Vec2d *sl, const Vec2d *sr)
    {
        if (!P.on()) return;
        Vec2d el = Vec2d{0.0, 0.0}, er = Vec2d{0.0, 0.0};
        if (P.sync) { el = sl[P.wave]; er = sr[P.wave + 1]; }
        Vec2d x[K], y[K];
#pragma unroll
        for (int k = 0; k < K; k++) { x[k] = before(k, el, P.lane); y[k] = after(k, er, P.lane); }
#pragma unroll
        for (int k = 0; k < K; k++) {
            const int p = P.pair(k);
            if (!P.own(k)) continue;
            double a[4] = {r[k][0], r[k][1], r[k][2], r[k][3]};
            const Vec2d e = Vec2d{du[k][0], du[k][1]}, o = Vec2d{du[k][2], du[k][3]};
            row<0, true>(R[k], x[k], e, o, a[0], a[1]);
            row<1, true>(R[k], e, o, y[k], a[2], a[3]);
            q0[p] = (T)(a[0] + a[2]);
            q1[p] = (T)(a[1] + a[3]);
        }
    }
};

template <typename T, int K>
__global__ void __launch_bounds__(kBottomNT) k_bottom(MGArgs mg, const int *inst_list, int zero_init0,
                                                      int final_update)
{
    constexpr int NP = kBottomNT * K;          // pairs of the first level
    constexpr int MC = kMaxCoarse;
    static_assert(kBottomNT >= MC, "the coarsest level needs one thread per cell");
    // cyclic reduction: D^{-1}, W, E and the right-hand side of every cell, in two buffers where
    // half the capacity is enough (a step then needs one barrier)
    __shared__ Vec2d cr[7 * MC];
    __shared__ Vec2d sl[kBottomNT / 64 + 1], sr[kBottomNT / 64 + 1];
    __shared__ long long Js[kMaxLevels];       // where the levels' operators begin
    // rhs and dU of the levels below the first, one level after the other; dU of the first behind
    __shared__ T q0[2 * NP], q1[2 * NP], d0[4 * NP], d1[4 * NP];
    const int inst = inst_list[blockIdx.x];
    const Inst1D &I = mg.insts[inst];
    T *base = reinterpret_cast<T *>(mg.mg);
    const int t = threadIdx.x;
    const int lb = I.lev0 + I.lbot;           // level-table index of the first bottom level
    const int nl = I.levc - lb + 1;           // levels handled here
    const double w = I.omega;
    const int nu1 = I.nu1, nu2 = I.nu2, N = I.N;
    double *const U0 = I.U;
    const double tau = I.tau;
    const bool finest = I.lbot == 0, update = finest && final_update;
    const Level1D &L0 = mg.levs[lb];
    const int n0 = L0.n;                      // level k of this kernel has n0 >> k cells
    const long long J0 = L0.J;
    T *const rhs0 = base + L0.rhs, *const dU0 = base + L0.dU;
    if (!active_of(mg, inst)) return;
    // pairs of overlap: 2 nu + 1 runs and the restriction each move information one cell
    const int g = max(nu1, nu2) + 1;
    // read once here: a later scalar read would be waited for with the LDS reads
    if (t < nl) Js[t] = mg.levs[lb + t].J;
    auto rows_of = [&](int k) -> const T * {
        const unsigned long long v = Js[k];
        const unsigned lo = __builtin_amdgcn_readfirstlane((int)(unsigned)v);
        const int hi = __builtin_amdgcn_readfirstlane((int)(v >> 32));
        return base + (((long long)hi << 32) | lo);
    };
    auto place = [&](int n, int k) { return PairPlace(n / 2, 0, n / 2, k, g, t, 0, kBottomNT / 64); };

    PairRows<T> nxt;                          // rows of the next level; the coarsest: one cell a thread
    PairRows<T> cur[1];
    PairLevel<T, 1> lev;
    auto fetch = [&](int k) {
        const int n = n0 >> k;
        const T *J = rows_of(k);
        if (k == nl - 1) {
            if (t < n) {
#pragma unroll
                for (int e = 0; e < 12; e++) nxt.j[e].x = J[e * (long long)n + t];
            }
        } else {
            const PairPlace P = place(n, 1);
            if (P.in(0)) load_rows(nxt, J, n, P.pair(0));
        }
    };

    // ---- down: pre-smoothing and restriction -------------------------------------------
    T r0[K][4];                               // rhs of the first level
    if (nl == 1) {
        __syncthreads();
        fetch(0);
    } else {
        PairRows<T> R[K];
        PairLevel<T, K> L;
        const PairPlace P = place(n0, K);
        const bool from_du = finest && !zero_init0;
#pragma unroll
        for (int k = 0; k < K; k++) {
            const int p = P.pair(k);
#pragma unroll
            for (int e = 0; e < 4; e++) { r0[k][e] = T(0); L.du[k][e] = 0.0; }
            if (P.in(k)) {
                load_rows(R[k], base + J0, n0, p);
                const auto x = ld2(rhs0 + 2 * p), y = ld2(rhs0 + n0 + 2 * p);
                r0[k][0] = x.x; r0[k][1] = y.x; r0[k][2] = x.y; r0[k][3] = y.y;
                if (from_du) {
                    const auto u = ld2(dU0 + 2 * p), v = ld2(dU0 + n0 + 2 * p);
                    L.du[k][0] = u.x; L.du[k][1] = v.x; L.du[k][2] = u.y; L.du[k][3] = v.y;
                }
            }
        }
        __syncthreads();                      // Js
        fetch(1);
        L.inverses(R, P);
#pragma unroll
        for (int k = 0; k < K; k++)
#pragma unroll
            for (int e = 0; e < 4; e++) L.r[k][e] = (double)r0[k][e];
        L.smooth(nu1, w, R, P, sl, sr);
        L.restrict_to(q0, q1, R, P, sl, sr);
#pragma unroll
        for (int k = 0; k < K; k++) {
            if (!P.own(k)) continue;
            st2(d0 + 2 * NP + 2 * P.pair(k), (T)L.du[k][0], (T)L.du[k][2]);
            st2(d1 + 2 * NP + 2 * P.pair(k), (T)L.du[k][1], (T)L.du[k][3]);
        }
        __syncthreads();
    }
    int qo = 0;                               // offset of level k in q0, q1, d0, d1
    for (int k = 1; k < nl - 1; k++) {
        const int n = n0 >> k;
        const PairPlace P = place(n, 1);
        const int c = qo + 2 * P.pair(0);
        cur[0] = nxt;
        fetch(k + 1);
#pragma unroll
        for (int e = 0; e < 4; e++) lev.r[0][e] = lev.du[0][e] = 0.0;
        if (P.in(0)) {
            const auto x = ld2(q0 + c), y = ld2(q1 + c);
            lev.r[0][0] = x.x; lev.r[0][1] = y.x; lev.r[0][2] = x.y; lev.r[0][3] = y.y;
        }
        lev.inverses(cur, P);
        lev.smooth(nu1, w, cur, P, sl, sr);
        lev.restrict_to(q0 + qo + n, q1 + qo + n, cur, P, sl, sr);
        if (P.own(0)) {
            st2(d0 + c, (T)lev.du[0][0], (T)lev.du[0][2]);
            st2(d1 + c, (T)lev.du[0][1], (T)lev.du[0][3]);
        }
        __syncthreads();
        qo += n;
    }

    // ---- coarsest: block parallel cyclic reduction ----------------------------------------------
    {
        const int n = n0 >> (nl - 1);
        const bool mine = t < n;
        double W[4] = {0, 0, 0, 0}, Dm[4] = {1, 0, 0, 1}, E[4] = {0, 0, 0, 0};
        double b0 = 0.0, b1 = 0.0;
        if (mine) {
#pragma unroll
            for (int e = 0; e < 4; e++) {
                // a row without the neighbour has no coupling to it: the steps below then need
                // no case for it (its W or E stays zero)
                W[e] = t > 0 ? (double)nxt.j[e].x : 0.0;
                Dm[e] = (double)nxt.j[4 + e].x;
                E[e] = t < n - 1 ? (double)nxt.j[8 + e].x : 0.0;
            }
            if (nl == 1) { b0 = -ld(rhs0, t); b1 = -ld(rhs0, n + (long long)t); }
            else { b0 = -(double)q0[qo + t]; b1 = -(double)q1[qo + t]; }
        }
        const bool two = n <= MC / 2;
        int buf = 0;
        for (int st = 1; st < n; st <<= 1) {
            if (!two) __syncthreads();
            Vec2d *const P = cr + buf;
            if (mine) {
                double Di[4];
                inv2(Dm, Di);
                P[0 * MC + t] = Vec2d{Di[0], Di[1]};
                P[1 * MC + t] = Vec2d{Di[2], Di[3]};
                P[2 * MC + t] = Vec2d{W[0], W[1]};
                P[3 * MC + t] = Vec2d{W[2], W[3]};
                P[4 * MC + t] = Vec2d{E[0], E[1]};
                P[5 * MC + t] = Vec2d{E[2], E[3]};
                P[6 * MC + t] = Vec2d{b0, b1};
            }
            __syncthreads();
            if (two) buf ^= MC / 2;
            if (mine) {
                struct Cell { Vec2d v[7]; };
                Cell l, h;                     // the cells at distance st before and after
                const int xl = t >= st ? t - st : t, xh = t + st < n ? t + st : t;
#pragma unroll
                for (int e = 0; e < 7; e++) { l.v[e] = P[e * MC + xl]; h.v[e] = P[e * MC + xh]; }
                // M <- a M', D <- D + a O', b <- b + a b', a = -M D'^{-1}
                auto fold = [&](double M[4], const Cell &c, int own, int oth) {
                    const double Bi[4] = {c.v[0].a, c.v[0].b, c.v[1].a, c.v[1].b};
                    const double Bm[4] = {c.v[own].a, c.v[own].b, c.v[own + 1].a, c.v[own + 1].b};
                    const double Bo[4] = {c.v[oth].a, c.v[oth].b, c.v[oth + 1].a, c.v[oth + 1].b};
                    double a[4], tm[4];
                    mul2(M, Bi, tm);
#pragma unroll
                    for (int e = 0; e < 4; e++) a[e] = -tm[e];
                    mul2(a, Bm, M);
                    mul2(a, Bo, tm);
#pragma unroll
                    for (int e = 0; e < 4; e++) Dm[e] = Dm[e] + tm[e];
                    b0 = b0 + (a[0] * c.v[6].a + a[1] * c.v[6].b);
                    b1 = b1 + (a[2] * c.v[6].a + a[3] * c.v[6].b);
                };
                fold(W, l, 2, 4);
                fold(E, h, 4, 2);
            }
        }
        if (mine) {
            double Di[4];
            inv2(Dm, Di);
            const double x0 = Di[0] * b0 + Di[1] * b1;
            const double x1 = Di[2] * b0 + Di[3] * b1;
            if (nl > 1) {
                d0[qo + t] = (T)x0;
                d1[qo + t] = (T)x1;
            } else if (update) {   // one-level hierarchy: the Newton update, eq. (14)
                U0[t] = U0[t] + tau * x0;
                U0[N + t] = U0[N + t] + tau * x1;
            } else {                          // the bottom is the coarsest level only
                dU0[t] = (T)x0;
                dU0[n + (long long)t] = (T)x1;
            }
        }
        __syncthreads();
    }
    if (nl == 1) return;

    // ---- up: prolongation and post-smoothing ------------------------------------------------
    auto climb = [&](int k) {                 // level k >= 1, its rows in cur; the child's dU at qo
        const int n = n0 >> k;
        const PairPlace P = place(n, 1);
        const int p = P.pair(0), c = qo - n + 2 * p;
        lev.inverses(cur, P);
#pragma unroll
        for (int e = 0; e < 4; e++) lev.r[0][e] = lev.du[0][e] = 0.0;
        if (P.in(0)) {
            const double p0 = (double)d0[qo + p], p1 = (double)d1[qo + p];
            const auto x = ld2(q0 + c), y = ld2(q1 + c), u = ld2(d0 + c), v = ld2(d1 + c);
            lev.r[0][0] = x.x; lev.r[0][1] = y.x; lev.r[0][2] = x.y; lev.r[0][3] = y.y;
            lev.du[0][0] = (double)u.x + p0;
            lev.du[0][1] = (double)v.x + p1;
            lev.du[0][2] = (double)u.y + p0;
            lev.du[0][3] = (double)v.y + p1;
        }
        __syncthreads();                      // windows read their neighbours' pairs of d0, d1 too
        lev.smooth(nu2, w, cur, P, sl, sr);
        if (P.own(0)) {
            st2(d0 + c, (T)lev.du[0][0], (T)lev.du[0][2]);
            st2(d1 + c, (T)lev.du[0][1], (T)lev.du[0][3]);
        }
        __syncthreads();
        qo -= n;
    };
    for (int k = nl - 2; k >= 2; k--) {       // the lowest level's rows are still in cur
        fetch(k - 1);
        climb(k);
        cur[0] = nxt;
    }
    PairRows<T> R[K];
    PairLevel<T, K> L;
    const PairPlace P = place(n0, K);
#pragma unroll
    for (int k = 0; k < K; k++)
        if (P.in(k)) load_rows(R[k], base + J0, n0, P.pair(k));
    if (nl > 2) climb(1);
    L.inverses(R, P);
#pragma unroll
    for (int k = 0; k < K; k++) {
        const int p = P.pair(k);
#pragma unroll
        for (int e = 0; e < 4; e++) { L.r[k][e] = (double)r0[k][e]; L.du[k][e] = 0.0; }
        if (P.in(k)) {
            const double p0 = (double)d0[p], p1 = (double)d1[p];
            const auto u = ld2(d0 + 2 * NP + 2 * p), v = ld2(d1 + 2 * NP + 2 * p);
            L.du[k][0] = (double)u.x + p0;
            L.du[k][1] = (double)v.x + p1;
            L.du[k][2] = (double)u.y + p0;
            L.du[k][3] = (double)v.y + p1;
        }
    }
    L.smooth(nu2, w, R, P, sl, sr);
#pragma unroll
    for (int k = 0; k < K; k++) {
        const int p = P.pair(k);
        if (!P.own(k)) continue;
        if (update) {
            double *U = U0 + 2 * p, *V = U0 + N + 2 * p;
            const auto u = ld2(U), v = ld2(V);
            st2(U, u.x + tau * L.du[k][0], u.y + tau * L.du[k][2]);
            st2(V, v.x + tau * L.du[k][1], v.y + tau * L.du[k][3]);
        } else {
            st2(dU0 + 2 * p, (T)L.du[k][0], (T)L.du[k][2]);
            st2(dU0 + n0 + 2 * p, (T)L.du[k][1], (T)L.du[k][3]);
        }
    }
}

// ---- levels above the bottom, several in one launch ----------------------------------------------
// Few cells in all (one channel, a handful of small ones): a launch per level costs its start, the
// chain of table reads and one wait for memory, 5 to 6 us, for under 1 us of smoothing.  Here one
// 256-thread workgroup takes up to kGroupLevels levels of a tile: the tile has a margin from which
// the levels' windows shrink (down) or grow (up), and everything the levels need is read at the
// start, the first level on all four wavefronts, the second on two, the third and fourth on one
// each.  MODE 0: pre-smoothing and restriction from the first level of the group to the child of its
// last; MODE 1: prolongation and post-smoothing back up to the first.
// Same arithmetic, in the same order, as a launch per level.

template <typename T, int MODE>
__global__ void __launch_bounds__(kGroupNT) k_group(MGArgs mg, const Tile *tiles, int zero_init, int final_update,
                                                    int src_out)
{
    constexpr int NW = kGroupNT / 64, CAP = 2 * 64 * NW;     // cells of the first level
    static_assert(NW == 4 && kGroupLevels == 4, "levels 1, 2 and 3 lie on wavefronts 0-1, 2 and 3");
    // rhs (down) and dU of the levels, level l's at offset CAP (2 - 2^(1-l))
    __shared__ T q0[2 * CAP], q1[2 * CAP], d0[2 * CAP], d1[2 * CAP];
    const Tile tl = tiles[blockIdx.x];
    const int t = threadIdx.x;
    const int inst = mg.levs[tl.lev].inst, n0 = mg.levs[tl.lev].n, top = mg.levs[tl.lev].l;
    const Inst1D &I = mg.insts[inst];
    const int nu = MODE == 0 ? I.nu1 : I.nu2;
    const Group1D G = group_window(max(I.nu1, I.nu2), I.lbot - top);
    const Level1D *const lev = mg.levs + tl.lev;             // of the group's levels and the child of its last
    // the wavefront's other level; none (level 0 again, unused) where the group is shorter
    const int wv = __builtin_amdgcn_readfirstlane(t >> 6), lw = wv < 2 ? 1 : wv;
    const bool other = lw < G.levels;
    const Level1D L0 = lev[0], L1 = lev[other ? lw : 0];
    const long long dUc = lev[G.levels].dU;
    const double w = I.omega, tau = I.tau;
    double *const U0 = I.U;
    const int N = I.N;
    if (!active_of(mg, inst)) return;
    T *const base = reinterpret_cast<T *>(mg.mg);
    const int s0 = tl.a - G.margin;                          // first cell of the window, level 0
    auto place = [&](int l) {
        const int org = (s0 >> l) / 2, np = (G.cells >> l) / 2;
        return PairPlace(np, max(0, -org), min(np, (n0 >> l) / 2 - org), 1, G.g, t, l < 2 ? 0 : l, l == 0 ? NW : l == 1 ? 2 : 1);
    };
    auto off = [&](int l) { return 2 * CAP - (2 * CAP >> l); };

    // ---- reads: level 0 in a, the wavefront's other level in b ---------------------------------
    PairRows<T> Ra[1], Rb[1];
    PairLevel<T, 1> A, B;
    auto read = [&](int l, const Level1D &V, bool there, PairRows<T> &R, PairLevel<T, 1> &L) {
        const PairPlace P = place(l);
        const int n = n0 >> l, p = (s0 >> l) / 2 + P.pair(0);
#pragma unroll
        for (int e = 0; e < 4; e++) L.r[0][e] = L.du[0][e] = 0.0;
        const T *const f = base + V.rhs + 2 * (long long)p;
        const T *const d = base + ((l == 0 ? src_out : 1) ? V.dUo : V.dU) + 2 * (long long)p;
        if (!there || !P.in(0)) return;
        load_rows(R, base + V.J, n, p);
        if (MODE == 1 || l == 0) {
            const auto x = ld2(f), y = ld2(f + n);
            L.r[0][0] = x.x; L.r[0][1] = y.x; L.r[0][2] = x.y; L.r[0][3] = y.y;
        }
        if (MODE == 1 || (l == 0 && !zero_init)) {
            const auto x = ld2(d), y = ld2(d + n);
            L.du[0][0] = x.x; L.du[0][1] = y.x; L.du[0][2] = x.y; L.du[0][3] = y.y;
        }
    };
    read(0, L0, true, Ra[0], A);
    read(lw, L1, other, Rb[0], B);
    auto store = [&](int l, PairLevel<T, 1> &L, const PairPlace &P) {
        if (!P.own(0)) return;
        st2(d0 + off(l) + 2 * P.pair(0), (T)L.du[0][0], (T)L.du[0][2]);
        st2(d1 + off(l) + 2 * P.pair(0), (T)L.du[0][1], (T)L.du[0][3]);
    };

    if (MODE == 0) {
        const PairPlace P0 = place(0), P1 = place(lw);
        A.inverses(Ra, P0);
        if (other) B.inverses(Rb, P1);
        A.smooth(nu, w, Ra, P0, nullptr, nullptr);
        A.restrict_to(q0 + off(1), q1 + off(1), Ra, P0, nullptr, nullptr);
        store(0, A, P0);
        __syncthreads();
        for (int l = 1; l < G.levels; l++) {
            if (lw == l) {
                if (P1.in(0)) {
                    const auto x = ld2(q0 + off(l) + 2 * P1.pair(0)), y = ld2(q1 + off(l) + 2 * P1.pair(0));
                    B.r[0][0] = x.x; B.r[0][1] = y.x; B.r[0][2] = x.y; B.r[0][3] = y.y;
                }
                B.smooth(nu, w, Rb, P1, nullptr, nullptr);
                B.restrict_to(q0 + off(l + 1), q1 + off(l + 1), Rb, P1, nullptr, nullptr);
                store(l, B, P1);
            }
            __syncthreads();
        }
        // the tile's own cells: dU of each level and the rhs of its child
        for (int l = 0; l < G.levels; l++) {
            const int m = G.margin >> l, n = n0 >> l, a = tl.a >> l, v = min(G.own >> l, n - a);
            T *du = base + ((l == 0 ? !src_out : 1) ? lev[l].dUo : lev[l].dU) + a, *f = base + lev[l + 1].rhs + a / 2;
            const int o = off(l) + m, c = off(l + 1) + m / 2;
            for (int i = t; i < v; i += kGroupNT) { du[i] = d0[o + i]; du[n + i] = d1[o + i]; }
            for (int i = t; i < v / 2; i += kGroupNT) { f[i] = q0[c + i]; f[n / 2 + i] = q1[c + i]; }
        }
    } else {
        const PairPlace P0 = place(0), P1 = place(lw);
        A.inverses(Ra, P0);
        if (other) B.inverses(Rb, P1);
        // dU of the child of the last level, cells of the window
        const int lc = G.levels, nc = n0 >> lc, sc = s0 >> lc;
        const T *f = base + dUc;
        for (int i = t; i < (G.cells >> lc); i += kGroupNT) {
            const bool in = sc + i >= 0 && sc + i < nc;
            d0[off(lc) + i] = in ? f[sc + i] : T(0);
            d1[off(lc) + i] = in ? f[nc + sc + i] : T(0);
        }
        __syncthreads();
        auto add_parent = [&](int l, PairLevel<T, 1> &L, const PairPlace &P) {
            if (!P.in(0)) return;
            const double c0 = (double)d0[off(l + 1) + P.pair(0)], c1 = (double)d1[off(l + 1) + P.pair(0)];
            L.du[0][0] = L.du[0][0] + c0;
            L.du[0][1] = L.du[0][1] + c1;
            L.du[0][2] = L.du[0][2] + c0;
            L.du[0][3] = L.du[0][3] + c1;
        };
        for (int l = G.levels - 1; l >= 1; l--) {
            if (lw == l) {
                add_parent(l, B, P1);
                B.smooth(nu, w, Rb, P1, nullptr, nullptr);
                store(l, B, P1);
            }
            __syncthreads();
        }
        add_parent(0, A, P0);
        A.smooth(nu, w, Ra, P0, nullptr, nullptr);
        const int c = 2 * P0.pair(0), j = s0 + c;            // cell in the window, in the level
        if (P0.own(0) && c >= G.margin && c < G.margin + G.own) {
            if (final_update) {                              // eq. (14)
                const auto u = ld2(U0 + j), v = ld2(U0 + N + j);
                st2(U0 + j, u.x + tau * A.du[0][0], u.y + tau * A.du[0][2]);
                st2(U0 + N + j, v.x + tau * A.du[0][1], v.y + tau * A.du[0][3]);
            } else {
                T *du = base + (src_out ? L0.dU : L0.dUo) + j;
                st2(du, (T)A.du[0][0], (T)A.du[0][2]);
                st2(du + n0, (T)A.du[0][1], (T)A.du[0][3]);
            }
        }
    }
}

// ---- Newton-SOR (section 5.1.1) ----------------------------------------------------------
// The reference solver of the paper's Table 2: each Newton step solves the regularised system on
// the grid itself by symmetric block SOR steps (eq. 19) until the l1 norm of the change of dU
// between two successive steps falls below a tolerance or a step limit is reached.  The
// multicolour step reuses the tiled smoother's structure (one symmetric step per launch, halo
// for one step) and reports the change per tile; a finalisation launch per Newton-SOR step sums
// it per instance (fixed order) and marks the instance done, after which the later steps of the
// same Newton step skip it.

template <typename T, int NB>
__global__ void __launch_bounds__(kTile) k_sor_mc(MGArgs mg, const Tile *tiles, int step, double *partial)
{
    const bool zero_init = step == 0;
    constexpr int HW = NB / 2;
    constexpr int C = NB == 5 ? 3 : 2;
    __shared__ double s0[kTile + 2 * HW], s1[kTile + 2 * HW];
    __shared__ double red[kTile / 64];
    const Tile tl = tiles[blockIdx.x];
    const Level1D L = mg.levs[tl.lev];
    const int t = threadIdx.x;
    if (L.nb != NB) return;
    const Inst1D &I = mg.insts[L.inst];
    const NewtonState *S = mg.state ? &mg.state[I.active_idx] : nullptr;
    T *base = reinterpret_cast<T *>(mg.mg);
    const int n = L.n, h = L.halo;
    const int j = tl.a - h + t;
    const bool in = j >= 0 && j < n;
    // step k reads dU (k even) or dUo (k odd) and writes the other buffer
    const long long src = (step & 1) ? L.dUo : L.dU, dst = (step & 1) ? L.dU : L.dUo;
    if (S && (!S->active || S->sor_done)) {
        // stopped: carry the iterate over to the buffer the next step reads
        if (S->active && !zero_init && in && t >= h && t < h + L.V) {
            base[dst + j] = base[src + j];
            base[dst + n + (long long)j] = base[src + n + (long long)j];
        }
        if (t == 0) partial[blockIdx.x] = 0.0;
        return;
    }
    double Jr[NB][4], D[4], r0 = 0.0, r1 = 0.0, du0 = 0.0, du1 = 0.0;
#pragma unroll
    for (int b = 0; b < NB; b++)
#pragma unroll
        for (int e = 0; e < 4; e++) Jr[b][e] = in ? ld(base + L.J, (b * 4 + e) * (long long)n + j) : 0.0;
    if (in) inv2(Jr[HW], D);
    else D[0] = D[1] = D[2] = D[3] = 0.0;
    if (in) {
        r0 = ld(base + L.rhs, j);
        r1 = ld(base + L.rhs, n + (long long)j);
        if (!zero_init) {
            du0 = ld(base + src, j);
            du1 = ld(base + src, n + (long long)j);
        }
    }
    const double old0 = du0, old1 = du1;
    s0[t + HW] = du0;
    s1[t + HW] = du1;
    if (t < HW) { s0[t] = 0.0; s1[t] = 0.0; s0[kTile + HW + t] = 0.0; s1[kTile + HW + t] = 0.0; }
    __syncthreads();
    const double w = I.omega;
    const int col = ((j % C) + C) % C;
    for (int hs = 0; hs < 2 * C; hs++) {
        const int c = hs < C ? hs : 2 * C - 1 - hs;
        if (in && col == c) {
            double a0 = r0, a1 = r1;
#pragma unroll
            for (int b = 0; b < NB; b++) {
                if (b == HW) continue;
                const double x0 = s0[t + b], x1 = s1[t + b];
                a0 = a0 + (Jr[b][0] * x0 + Jr[b][1] * x1);
                a1 = a1 + (Jr[b][2] * x0 + Jr[b][3] * x1);
            }
            const double t0 = D[0] * a0 + D[1] * a1;
            const double t1 = D[2] * a0 + D[3] * a1;
            du0 = (1.0 - w) * du0 - w * t0;
            du1 = (1.0 - w) * du1 - w * t1;
            s0[t + HW] = du0;
            s1[t + HW] = du1;
        }
        __syncthreads();
    }
    const bool valid = in && t >= h && t < h + L.V;
    double v = 0.0;
    if (valid) {
        base[dst + j] = (T)du0;
        base[dst + n + (long long)j] = (T)du1;
        v = fabs((double)(T)du0 - old0) + fabs((double)(T)du1 - old1);
    }
    for (int off = 32; off > 0; off >>= 1) v += __shfl_down(v, off, 64);
    if ((t & 63) == 0) red[t >> 6] = v;
    __syncthreads();
    if (t == 0) {
        double sum = 0.0;
        for (int k = 0; k < kTile / 64; k++) sum += red[k];
        partial[blockIdx.x] = sum;
    }
}

// per instance: the change of this Newton-SOR step from its tiles' partial sums
__global__ void __launch_bounds__(64) k_sor_finalize(const Inst1D *insts, int ninst, NewtonState *state,
                                                     const double *partial, double tol)
{
    const int b = blockIdx.x;
    if (b >= ninst) return;
    const Inst1D &I = insts[b];
    NewtonState &S = state[I.active_idx];
    if (!S.active || S.sor_done) return;
    double v = 0.0;
    for (int k = threadIdx.x; k < I.sor_tiles; k += 64) v += partial[I.sor_tile0 + k];
    for (int off = 32; off > 0; off >>= 1) v += __shfl_down(v, off, 64);
    if (threadIdx.x == 0 && v < tol) S.sor_done = 1;
}

// The lexicographic symmetric step (forward then backward sweep, eq. 19) of one instance per
// workgroup, with its own stopping test.  The sweep is sequential (a cell uses the new values of
// the cells before it), so one lane performs it, reading from LDS: the workgroup stages it in
// chunks of kLexChunk cells in sweep order (the off-diagonal blocks, the inverse of the diagonal
// block -- formed by the loading lanes, not on the sweep's critical path -- the right-hand side
// and the current dU, plus the dU of HW cells ahead), three wavefronts loading the next chunk
// into the other buffer while the first lane sweeps the current one.  The sweeping lane keeps
// the new dU of the last HW cells in registers (the cells behind the next one, also across a
// chunk edge), and each swept chunk is written back before its buffer is refilled.  The change
// norm is summed in cell order by one lane from per-cell terms formed in parallel.  Every value
// and every sum is formed as the sequential sweep over global memory forms it, so the results
// are the same bit for bit.
constexpr int kLexChunk = 256;

template <typename T, int NB>
__device__ __forceinline__ void lex_load_chunk(const T *base, const Level1D &L, int n, int k, bool fwd, int t0,
                                               int nt, double (*bJ)[kLexChunk + NB - 1],
                                               double (*bR)[kLexChunk + NB - 1], double (*bU)[kLexChunk + NB - 1])
{
    constexpr int HW = NB / 2;
    for (int sl = HW + t0; sl < kLexChunk + 2 * HW; sl += nt) {   // the chunk and HW cells ahead
        const int q = k * kLexChunk - HW + sl;
        if (q >= n) continue;
        const int j = fwd ? q : n - 1 - q;
        bU[0][sl] = ld(base + L.dU, j);
        bU[1][sl] = ld(base + L.dU, n + (long long)j);
        if (sl < HW + kLexChunk) {
            bR[0][sl] = ld(base + L.rhs, j);
            bR[1][sl] = ld(base + L.rhs, n + (long long)j);
            double Jd[4], D[4];
#pragma unroll
            for (int e = 0; e < NB * 4; e++) {
                const double v = ld(base + L.J, e * (long long)n + j);
                if (e >= HW * 4 && e < HW * 4 + 4) Jd[e - HW * 4] = v;
                else bJ[e][sl] = v;
            }
            inv2(Jd, D);   // the diagonal block's slots hold its inverse
#pragma unroll
            for (int e = 0; e < 4; e++) bJ[HW * 4 + e][sl] = D[e];
        }
    }
}

template <typename T, int NB>
__global__ void __launch_bounds__(256) k_sor_lex(MGArgs mg, int zero_init, double tol)
{
    constexpr int HW = NB / 2, SL = kLexChunk + 2 * HW;
    __shared__ double bJ[2][NB * 4][SL], bR[2][2][SL], bU[2][2][SL];
    const Inst1D &I = mg.insts[blockIdx.x];
    NewtonState *S = mg.state ? &mg.state[I.active_idx] : nullptr;
    if (S && (!S->active || S->sor_done)) return;
    const Level1D L = mg.levs[I.lev0];
    if (L.nb != NB) return;
    T *base = reinterpret_cast<T *>(mg.mg);
    const int n = L.n, t = threadIdx.x;
    const double w = I.omega;
    // keep the iterate before this step in aux (zero at the first step of a Newton step)
    for (int j = t; j < n; j += blockDim.x) {
        const double d0 = zero_init ? 0.0 : ld(base + L.dU, j);
        const double d1 = zero_init ? 0.0 : ld(base + L.dU, n + (long long)j);
        base[L.aux + j] = (T)d0;
        base[L.aux + n + (long long)j] = (T)d1;
        if (zero_init) { base[L.dU + j] = (T)0.0; base[L.dU + n + (long long)j] = (T)0.0; }
    }
    __syncthreads();
    const int nch = (n + kLexChunk - 1) / kLexChunk;
    for (int pass = 0; pass < 2; pass++) {
        const bool fwd = pass == 0;
        lex_load_chunk<T, NB>(base, L, n, 0, fwd, t, blockDim.x, bJ[0], bR[0], bU[0]);
        __syncthreads();
        // lane 0: the new dU of the last HW cells swept, p[m] at m + 1 positions behind the next
        double p0[HW], p1[HW];
#pragma unroll
        for (int m = 0; m < HW; m++) p0[m] = p1[m] = 0.0;
        for (int k = 0; k < nch; k++) {
            const int b = k & 1;
            if (t == 0) {
                const int q1 = min(n, (k + 1) * kLexChunk);
                // unrolled: the loads of the next cells issue while this cell's chain runs
#pragma unroll 4
                for (int q = k * kLexChunk; q < q1; q++) {
                    const int j = fwd ? q : n - 1 - q;
                    const int sl = q - k * kLexChunk + HW;
                    double a0 = bR[b][0][sl], a1 = bR[b][1][sl];
#pragma unroll
                    for (int bb = 0; bb < NB; bb++) {
                        const int i = j + bb - HW;
                        if (bb == HW || i < 0 || i >= n) continue;
                        const int off = fwd ? bb - HW : HW - bb;   // position of cell i relative to q
                        double x0, x1;
                        if (off < 0) { x0 = p0[-off - 1]; x1 = p1[-off - 1]; }   // swept: its new value
                        else { x0 = bU[b][0][sl + off]; x1 = bU[b][1][sl + off]; }
                        a0 = a0 + (bJ[b][bb * 4 + 0][sl] * x0 + bJ[b][bb * 4 + 1][sl] * x1);
                        a1 = a1 + (bJ[b][bb * 4 + 2][sl] * x0 + bJ[b][bb * 4 + 3][sl] * x1);
                    }
                    const double D0 = bJ[b][HW * 4 + 0][sl], D1 = bJ[b][HW * 4 + 1][sl];
                    const double D2 = bJ[b][HW * 4 + 2][sl], D3 = bJ[b][HW * 4 + 3][sl];
                    const double t0 = D0 * a0 + D1 * a1;
                    const double t1 = D2 * a0 + D3 * a1;
                    const double d0 = bU[b][0][sl], d1 = bU[b][1][sl];
                    // rounded to the storage type, as the value a sweep over global memory reads back
                    const double n0 = (double)(T)((1.0 - w) * d0 - w * t0);
                    const double n1 = (double)(T)((1.0 - w) * d1 - w * t1);
                    bU[b][0][sl] = n0;
                    bU[b][1][sl] = n1;
#pragma unroll
                    for (int m = HW - 1; m > 0; m--) { p0[m] = p0[m - 1]; p1[m] = p1[m - 1]; }
                    p0[0] = n0;
                    p1[0] = n1;
                }
            } else if (t >= 64 && k + 1 < nch) {
                lex_load_chunk<T, NB>(base, L, n, k + 1, fwd, t - 64, blockDim.x - 64, bJ[b ^ 1], bR[b ^ 1], bU[b ^ 1]);
            }
            __syncthreads();
            for (int sl = HW + t; sl < HW + kLexChunk; sl += blockDim.x) {   // write the swept chunk back
                const int q = k * kLexChunk - HW + sl;
                if (q >= n) continue;
                const int j = fwd ? q : n - 1 - q;
                base[L.dU + j] = (T)bU[b][0][sl];
                base[L.dU + n + (long long)j] = (T)bU[b][1][sl];
            }
            __syncthreads();
        }
    }
    // l1 norm of the change over the whole step, cells in order, components interleaved
    double v = 0.0;
    for (int k = 0; k < nch; k++) {
        for (int c = t; c < kLexChunk; c += blockDim.x) {
            const int j = k * kLexChunk + c;
            if (j < n) {
                bR[0][0][c] = fabs(ld(base + L.dU, j) - ld(base + L.aux, j));
                bR[0][1][c] = fabs(ld(base + L.dU, n + (long long)j) - ld(base + L.aux, n + (long long)j));
            }
        }
        __syncthreads();
        if (t == 0) {
            const int c1 = min(kLexChunk, n - k * kLexChunk);
            for (int c = 0; c < c1; c++) {
                v += bR[0][0][c];
                v += bR[0][1][c];
            }
        }
        __syncthreads();
    }
    if (t == 0 && S && v < tol) S->sor_done = 1;
}

// eq. (14) after the Newton-SOR steps: U <- U + tau dU on level 0 of every active instance
template <typename T>
__global__ void __launch_bounds__(kTile) k_update1d(MGArgs mg, const Tile *tiles, int from_out)
{
    const Tile tl = tiles[blockIdx.x];
    const Inst1D &I = mg.insts[tl.lev];
    if (mg.state && !mg.state[I.active_idx].active) return;
    const Level1D L = mg.levs[I.lev0];
    const T *base = reinterpret_cast<const T *>(mg.mg);
    const int j = tl.a + threadIdx.x;
    if (j >= I.N) return;
    const long long d = from_out ? L.dUo : L.dU;
    I.U[j] = I.U[j] + I.tau * ld(base + d, j);
    I.U[I.N + j] = I.U[I.N + j] + I.tau * ld(base + d, L.n + (long long)j);
}

// Initial cell averages of a grid from the solution on the grid with half as many cells
// (Appendix A, eq. A.1-A.2), both components; one thread per coarse cell.  Interior cells use
// eq. (A.2); the first and last coarse cells average, over their two halves, the quadratic
// (A.1) of the neighbouring interior cell.
__global__ void k_interp_a2(const double *Uc, int nc, double *Uf)
{
    const int j = blockIdx.x * blockDim.x + threadIdx.x;
    const int c = blockIdx.y;
    if (j >= nc) return;
    const double *u = Uc + (long long)c * nc;
    double *v = Uf + (long long)c * 2 * nc;
    if (j >= 1 && j <= nc - 2) {
        v[2 * j] = u[j - 1] / 8.0 + u[j] - u[j + 1] / 8.0;
        v[2 * j + 1] = -u[j - 1] / 8.0 + u[j] + u[j + 1] / 8.0;
        return;
    }
    const int k = j == 0 ? 1 : nc - 2;          // centre of the quadratic used
    const double a = (u[k + 1] - u[k - 1]) / 2.0;
    const double b = (u[k - 1] - 2.0 * u[k] + u[k + 1]) / 2.0;
#pragma unroll
    for (int half = 0; half < 2; half++) {
        // this half of cell j spans xi in [lo, hi], xi = (x - x_k) / dx of the coarse grid
        const double lo = (double)(j - k) - 0.5 + 0.5 * half, hi = lo + 0.5;
        const double m1 = (lo + hi) / 2.0;
        const double m2 = (lo * lo + lo * hi + hi * hi) / 3.0;
        v[2 * j + half] = u[k] + a * m1 + b * (m2 - 1.0 / 12.0);
    }
}

hipError_t launch_sor_mc(const MGArgs &mg, const Tile *tiles, int ntiles, int nb_max, int step,
                         double *partial, int prec, hipStream_t s)
{
    if (ntiles == 0) return hipSuccess;
    if (prec == NMG_FP32_MG) {
        hipLaunchKernelGGL((k_sor_mc<float, 3>), dim3(ntiles), dim3(kTile), 0, s, mg, tiles, step, partial);
        if (nb_max == 5)
            hipLaunchKernelGGL((k_sor_mc<float, 5>), dim3(ntiles), dim3(kTile), 0, s, mg, tiles, step, partial);
    } else {
        hipLaunchKernelGGL((k_sor_mc<double, 3>), dim3(ntiles), dim3(kTile), 0, s, mg, tiles, step, partial);
        if (nb_max == 5)
            hipLaunchKernelGGL((k_sor_mc<double, 5>), dim3(ntiles), dim3(kTile), 0, s, mg, tiles, step, partial);
    }
    return hipGetLastError();
}

hipError_t launch_sor_finalize(const Inst1D *insts, int ninst, NewtonState *state, const double *partial,
                               double tol, hipStream_t s)
{
    hipLaunchKernelGGL(k_sor_finalize, dim3(ninst), dim3(64), 0, s, insts, ninst, state, partial, tol);
    return hipGetLastError();
}

hipError_t launch_sor_lex(const MGArgs &mg, int ninst, int nb_max, int zero_init, double tol, int prec,
                          hipStream_t s)
{
    const dim3 grid(ninst);   // one workgroup per instance
    if (prec == NMG_FP32_MG) {
        hipLaunchKernelGGL((k_sor_lex<float, 3>), grid, dim3(256), 0, s, mg, zero_init, tol);
        if (nb_max == 5) hipLaunchKernelGGL((k_sor_lex<float, 5>), grid, dim3(256), 0, s, mg, zero_init, tol);
    } else {
        hipLaunchKernelGGL((k_sor_lex<double, 3>), grid, dim3(256), 0, s, mg, zero_init, tol);
        if (nb_max == 5) hipLaunchKernelGGL((k_sor_lex<double, 5>), grid, dim3(256), 0, s, mg, zero_init, tol);
    }
    return hipGetLastError();
}

hipError_t launch_update1d(const MGArgs &mg, const Tile *tiles, int ntiles, int from_out, int prec, hipStream_t s)
{
    if (ntiles == 0) return hipSuccess;
    if (prec == NMG_FP32_MG)
        hipLaunchKernelGGL(k_update1d<float>, dim3(ntiles), dim3(kTile), 0, s, mg, tiles, from_out);
    else hipLaunchKernelGGL(k_update1d<double>, dim3(ntiles), dim3(kTile), 0, s, mg, tiles, from_out);
    return hipGetLastError();
}

hipError_t launch_interp_a2(const double *Uc, int nc, double *Uf, hipStream_t s)
{
    hipLaunchKernelGGL(k_interp_a2, dim3((nc + 255) / 256, 2), dim3(256), 0, s, Uc, nc, Uf);
    return hipGetLastError();
}

template <typename S, typename D>
__global__ void k_convert(const S *src, D *dst, long long n)
{
    for (long long i = blockIdx.x * (long long)blockDim.x + threadIdx.x; i < n;
         i += (long long)gridDim.x * blockDim.x)
        dst[i] = (D)src[i];
}

// ---- launchers ---------------------------------------------------------------------------

hipError_t launch_coarsen1d(const MGArgs &mg, const Tile *tiles, int ntiles, int prec, hipStream_t s)
{
    if (ntiles == 0) return hipSuccess;
    if (prec == NMG_FP32_MG)
        hipLaunchKernelGGL(k_coarsen<float>, dim3(ntiles), dim3(kTile), 0, s, mg, tiles);
    else
        hipLaunchKernelGGL(k_coarsen<double>, dim3(ntiles), dim3(kTile), 0, s, mg, tiles);
    return hipGetLastError();
}

template <typename T>
static void launch_bottom_t(const MGArgs &mg, const int *inst_list, int n, int zero_init0, int final_update,
                            int nt, hipStream_t s)
{
    // nt = half the cells of the largest first level: one pair a thread up to 1024 cells, else two
    if (nt <= kBottomNT)
        hipLaunchKernelGGL((k_bottom<T, 1>), dim3(n), dim3(kBottomNT), 0, s, mg, inst_list, zero_init0, final_update);
    else
        hipLaunchKernelGGL((k_bottom<T, 2>), dim3(n), dim3(kBottomNT), 0, s, mg, inst_list, zero_init0, final_update);
}

hipError_t launch_bottom(const MGArgs &mg, const int *inst_list, int n, int zero_init0, int final_update,
                         int prec, int nt, hipStream_t s)
{
    if (n == 0) return hipSuccess;
    if (nt != 256 && nt != 512 && nt != 1024) return hipErrorInvalidValue;
    if (prec == NMG_FP32_MG) launch_bottom_t<float>(mg, inst_list, n, zero_init0, final_update, nt, s);
    else launch_bottom_t<double>(mg, inst_list, n, zero_init0, final_update, nt, s);
    return hipGetLastError();
}

template <typename T, int NB, int TW>
static void launch_smooth_w(const MGArgs &mg, const Tile *tiles, int ntiles, int mode, int zero_init,
                            int final_update, int src_out, int reverse, hipStream_t s)
{
    if (mode == 0)
        hipLaunchKernelGGL((k_smooth<T, NB, 0, TW>), dim3(ntiles), dim3(TW), 0, s, mg, tiles, zero_init,
                           final_update, src_out, reverse);
    else if (mode == 1)
        hipLaunchKernelGGL((k_smooth<T, NB, 1, TW>), dim3(ntiles), dim3(TW), 0, s, mg, tiles, zero_init,
                           final_update, src_out, reverse);
    else
        hipLaunchKernelGGL((k_smooth<T, NB, 2, TW>), dim3(ntiles), dim3(TW), 0, s, mg, tiles, zero_init,
                           final_update, src_out, reverse);
}

template <typename T, int NB>
static void launch_smooth_t(const MGArgs &mg, const Tile *tiles, int ntiles, int mode, int zero_init,
                            int final_update, int src_out, int tile, int reverse, hipStream_t s)
{
    if (tile == kSmoothTileMax)
        launch_smooth_w<T, NB, kSmoothTileMax>(mg, tiles, ntiles, mode, zero_init, final_update, src_out, reverse, s);
    else
        launch_smooth_w<T, NB, kSmoothTile>(mg, tiles, ntiles, mode, zero_init, final_update, src_out, reverse, s);
}

hipError_t launch_smooth1d(const MGArgs &mg, const Tile *tiles, int ntiles, int nb_mask, int mode,
                           int zero_init, int final_update, int src_out, int prec, int tile, int reverse, hipStream_t s)
{
    if (ntiles == 0) return hipSuccess;
    if (tile != kSmoothTile && tile != kSmoothTileMax) return hipErrorInvalidValue;
    if (prec == NMG_FP32_MG) {
        if (nb_mask & 1) launch_smooth_t<float, 3>(mg, tiles, ntiles, mode, zero_init, final_update, src_out, tile, reverse, s);
        if (nb_mask & 2) launch_smooth_t<float, 5>(mg, tiles, ntiles, mode, zero_init, final_update, src_out, tile, reverse, s);
    } else {
        if (nb_mask & 1) launch_smooth_t<double, 3>(mg, tiles, ntiles, mode, zero_init, final_update, src_out, tile, reverse, s);
        if (nb_mask & 2) launch_smooth_t<double, 5>(mg, tiles, ntiles, mode, zero_init, final_update, src_out, tile, reverse, s);
    }
    return hipGetLastError();
}

hipError_t launch_group1d(const MGArgs &mg, const Tile *tiles, int ntiles, int mode, int zero_init, int final_update,
                          int src_out, int prec, hipStream_t s)
{
    if (ntiles == 0) return hipSuccess;
    const dim3 g(ntiles), b(kGroupNT);
    if (prec == NMG_FP32_MG) {
        if (mode == 0) hipLaunchKernelGGL((k_group<float, 0>), g, b, 0, s, mg, tiles, zero_init, final_update, src_out);
        else hipLaunchKernelGGL((k_group<float, 1>), g, b, 0, s, mg, tiles, zero_init, final_update, src_out);
    } else {
        if (mode == 0) hipLaunchKernelGGL((k_group<double, 0>), g, b, 0, s, mg, tiles, zero_init, final_update, src_out);
        else hipLaunchKernelGGL((k_group<double, 1>), g, b, 0, s, mg, tiles, zero_init, final_update, src_out);
    }
    return hipGetLastError();
}

hipError_t launch_convert(const void *src, int src_prec, void *dst, int dst_prec, long long n,
                          hipStream_t s)
{
    if (n == 0) return hipSuccess;
    int blocks = (int)((n + 255) / 256);
    if (blocks > 4096) blocks = 4096;
    if (src_prec == NMG_FP64 && dst_prec == NMG_FP64)
        hipLaunchKernelGGL((k_convert<double, double>), dim3(blocks), dim3(256), 0, s, (const double *)src, (double *)dst, n);
    else if (src_prec == NMG_FP64)
        hipLaunchKernelGGL((k_convert<double, float>), dim3(blocks), dim3(256), 0, s, (const double *)src, (float *)dst, n);
    else if (dst_prec == NMG_FP64)
        hipLaunchKernelGGL((k_convert<float, double>), dim3(blocks), dim3(256), 0, s, (const float *)src, (double *)dst, n);
    else
        hipLaunchKernelGGL((k_convert<float, float>), dim3(blocks), dim3(256), 0, s, (const float *)src, (float *)dst, n);
    return hipGetLastError();
}

}  // namespace nmg
