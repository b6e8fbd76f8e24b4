// 2D finite-volume residual (section 4.1, eq. 20) with characteristic WENO3, Gauss quadrature
// along faces and the tensor Gauss source, and its finite-difference Jacobian on the cross
// stencil of eq. (21) (J9) or the full 21-cell stencil (J21), for gfx950.
//
// The arithmetic is that of the formulas in their printed order, without FMA contraction and
// with correctly rounded division and square root, so every face state, flux and residual is
// reproducible bit for bit; with the 1e-6 perturbation of the 2D Jacobian anything less would
// be amplified a million times.
//
// Work sharing.  The residual of cell (i, j) is assembled from 36 characteristic face states
// (x faces on rows j-1..j+1, y faces on columns i-1..i+1, both sides of the four faces of the
// cell and the inner states of the next faces out, which the source's cubics need).  A face state
// depends only on three consecutive cells of its line, so a 32x8 tile computes every face state
// its cells use once, into LDS tables, then the flux through every face once, and each cell assembles
// its residual from them.  For the Jacobian a perturbation of cell p changes only the face states whose three cells include p, and
// a face state perturbed in one of its cells serves every row that has it: the interior kernel's
// tables hold each state with each of its three cells raised, component by component, and a row (at
// least two cells inside the grid, so without a ghost in its residual) re-forms only the fluxes
// and depths that the perturbed cell reaches.  The values equal a full re-evaluation of the
// perturbed local residual bit for bit.  Rows within two cells of a side, whose ghosts also follow
// the perturbed cell, list the states that do and re-form those.
//
// Surface variant (recon = NMG_RECON_SURFACE, template flag SURF of the state accessors): the
// reconstructions act on (eta, hu, hv), eta = h + zbar (zbar the cell average of b), in the
// characteristic basis of the two cells' (h, hu, hv); a face Gauss point's depth is eta minus b
// there; ghosts that copy a cell's depth copy its surface; each Gauss line's source takes the
// split form -g [int (eta_h - eta_ij) b_x + eta_ij (b_+ - b_-) - (b_+^2 - b_-^2) / 2].  Still
// water then has a zero residual to rounding on any bottom.
//
// Register discipline: every helper is force-inlined and passes values as small structs by
// value, indexed only by compile-time constants; boundary data of a side is selected by
// comparisons, never by a runtime array index.  The kernels keep their state in registers and
// LDS: no calls, no generic pointers into private memory.
#include "nmg_common.h"

namespace nmg {

constexpr int kTX = 32, kTY = 8;                       // tile of cells
constexpr int kSX = kTX + 4, kSY = kTY + 4;            // staged state (halo 2)
constexpr int kBorderNT = 64;                          // threads of a border-kernel workgroup
constexpr int kSlots = 36;                             // face states of one local residual

// Every helper is callable from host code too, so that a CPU build can replay the kernels' per-row
// arithmetic; NMG2D_CHECK is a bounds-check hook on staged and table reads for such a build.
#define NMG2D_INL __host__ __device__ __forceinline__
#ifndef NMG2D_CHECK
#define NMG2D_CHECK(cond) ((void)0)
#endif

struct V3 { double c[3]; };
struct H2 { double g[2]; };            // a depth at the two Gauss points of a face

// Division and square root rounded as IEEE 754 asks, for operands far from the overflow and denormal
// limits (depths, smoothness indicators, wave speeds): the reciprocal refined by two Newton-Raphson
// steps, the quotient corrected once by its residual (Markstein), and Goldschmidt's square root with
// two residual corrections.  The compiler's sequences are these with range scaling and special cases
// around them, which cost about a third of a quotient; and quotients of one divisor share its
// reciprocal here.  A zero or negative depth still gives a non-finite result.
struct Recip {
    double b, r;
    NMG2D_INL explicit Recip(double d) : b(d)
    {
#ifdef __HIP_DEVICE_COMPILE__
        r = __builtin_amdgcn_rcp(d);
        r = fma(fma(-d, r, 1.0), r, r);
        r = fma(fma(-d, r, 1.0), r, r);
#else
        r = 0.0;
#endif
    }
    NMG2D_INL double of(double a) const      // a / b
    {
#ifdef __HIP_DEVICE_COMPILE__
        const double q = a * r;
        return fma(fma(-b, q, a), r, q);
#else
        return a / b;
#endif
    }
};

NMG2D_INL double sqrt2(double a)
{
#ifdef __HIP_DEVICE_COMPILE__
    const double r = __builtin_amdgcn_rsq(a);
    double g = a * r, h = r * 0.5;
    const double e = fma(-h, g, 0.5);
    g = fma(g, e, g);
    h = fma(h, e, h);
    double d = fma(-g, g, a);
    g = fma(d, h, g);
    d = fma(-g, g, a);
    return fma(d, h, g);
#else
    return sqrt(a);
#endif
}

// The minus state's reconstruction: from cell u0 to the face on the side of up.  The plus state's is
// the mirror image, the same operations on the cells in the opposite order.
NMG2D_INL double weno_m2(double um, double u0, double up)
{
    double c0 = 0.5 * u0 + 0.5 * up;
    double c1 = -0.5 * um + 1.5 * u0;
    double b0 = (up - u0) * (up - u0);
    double b1 = (u0 - um) * (u0 - um);
    double a0 = Recip((kZeta + b0) * (kZeta + b0)).of(2.0 / 3.0);
    double a1 = Recip((kZeta + b1) * (kZeta + b1)).of(1.0 / 3.0);
    const Recip sum(a0 + a1);
    return sum.of(a0) * c0 + sum.of(a1) * c1;
}

// Characteristic WENO3 state of cell S1 at the face it shares with S2, from three consecutive cells
// of a line in either order (S0, S1, S2 along the line give the minus state of the face between S1 and
// S2, against it the plus state); components (depth, momentum along the line, momentum across it).
// The basis is the eigensystem of the face-normal flux Jacobian at the mean of the face's two cells.
// SURF: the projection acts on the surfaces S_q.c[0] + z_q (z_q the cell average of b), the
// basis on the depths.
template <bool SURF>
NMG2D_INL V3 face_state_line(const V3 &S0, const V3 &S1, const V3 &S2, double g, double z0 = 0.0, double z1 = 0.0,
                             double z2 = 0.0)
{
    const double h = 0.5 * (S1.c[0] + S2.c[0]);
    const Recip rh(h);
    const double un = rh.of(0.5 * (S1.c[1] + S2.c[1]));
    const double ut = rh.of(0.5 * (S1.c[2] + S2.c[2]));
    const double cc = sqrt2(g * h);
    const double i2c = Recip(2.0 * cc).of(1.0);
    const double la = (un + cc) * i2c, lb = -(un - cc) * i2c;
    double w[3];
#pragma unroll
    for (int f = 0; f < 3; f++) {
        double W[3];
#pragma unroll
        for (int q = 0; q < 3; q++) {
            const V3 &Sq = q == 0 ? S0 : (q == 1 ? S1 : S2);
            const double e = SURF ? Sq.c[0] + (q == 0 ? z0 : (q == 1 ? z1 : z2)) : Sq.c[0];
            W[q] = f == 0 ? la * e + -i2c * Sq.c[1] : (f == 1 ? -ut * e + Sq.c[2] : lb * e + i2c * Sq.c[1]);
        }
        w[f] = weno_m2(W[0], W[1], W[2]);
    }
    V3 out;
    out.c[0] = w[0] + w[2];
    out.c[1] = (un - cc) * w[0] + (un + cc) * w[2];
    out.c[2] = ut * w[0] + w[1] + ut * w[2];
    return out;
}

template <int DIR>
NMG2D_INL V3 flux2(const V3 &U, double g)
{
    const double h = U.c[0];
    const Recip rh(h);
    const double u = rh.of(U.c[1]);
    const double v = rh.of(U.c[2]);
    V3 F;
    if (DIR == 0) {
        F.c[0] = U.c[1];
        F.c[1] = U.c[1] * u + 0.5 * g * h * h;
        F.c[2] = U.c[1] * v;
    } else {
        F.c[0] = U.c[2];
        F.c[1] = U.c[2] * u;
        F.c[2] = U.c[2] * v + 0.5 * g * h * h;
    }
    return F;
}

template <int DIR>
NMG2D_INL V3 llf2(const V3 &UL, const V3 &UR, double g)
{
    const V3 FL = flux2<DIR>(UL, g);
    const V3 FR = flux2<DIR>(UR, g);
    const double unL = Recip(UL.c[0]).of(UL.c[1 + DIR]), unR = Recip(UR.c[0]).of(UR.c[1 + DIR]);
    const double sL = fabs(unL) + sqrt2(g * UL.c[0]);
    const double sR = fabs(unR) + sqrt2(g * UR.c[0]);
    const double a = sL > sR ? sL : sR;
    V3 F;
#pragma unroll
    for (int c = 0; c < 3; c++) F.c[c] = 0.5 * (FL.c[c] + FR.c[c] - a * (UR.c[c] - UL.c[c]));
    return F;
}

// The quadratic through three face averages at the Gauss point G (0: lower, 1: upper) of the
// face (its curvature term is zero there): V0 + t (Vp - Vm) / 2, t = -+1/(2 sqrt 3).
template <int G>
NMG2D_INL V3 gauss_pt2(const V3 &Vm, const V3 &V0, const V3 &Vp)
{
    const double t = G == 0 ? -1.0 / (2.0 * sqrt(3.0)) : 1.0 / (2.0 * sqrt(3.0));
    V3 P;
#pragma unroll
    for (int c = 0; c < 3; c++) {
        const double slope = (Vp.c[c] - Vm.c[c]) * 0.5;
        P.c[c] = V0.c[c] + t * slope;
    }
    return P;
}

// Lagrange weight of node K (nodes -3/2, -1/2, 1/2, 3/2) of the cubic at the Gauss point Q
// (0: -1/(2 sqrt 3), 1: +1/(2 sqrt 3)), as the product over the other nodes in node order
template <int Q, int K>
NMG2D_INL double cubic_w2()
{
    const double x = Q == 0 ? -1.0 / (2.0 * sqrt(3.0)) : 1.0 / (2.0 * sqrt(3.0));
    const double t[4] = {-1.5, -0.5, 0.5, 1.5};
    double v = 1.0;
#pragma unroll
    for (int m = 0; m < 4; m++)
        if (m != K) v *= (x - t[m]) / (t[K] - t[m]);
    return v;
}

template <int Q>
NMG2D_INL double cubic_at2(double h0, double h1, double h2, double h3)
{
    return cubic_w2<Q, 0>() * h0 + cubic_w2<Q, 1>() * h1 + cubic_w2<Q, 2>() * h2 + cubic_w2<Q, 3>() * h3;
}

// Local residual R_ij of eq. (20) from its 36 face states.  FS::get<DIR, W, K, A>() gives the
// state of side W of the face between cells A and A+1 (relative to the row cell along the
// direction DIR) on the line at offset K across it.  bx, by: the cell's bottom slopes at its 2x2
// Gauss points ([beta][gamma], beta the y point).
// hm, hp: the first component of the two states at the Gauss points (the depth, or the surface
// in the surface variant, whose depths are then those minus b0, b1, b at the two points)
template <int DIR, int A, class FS>
NMG2D_INL V3 face_flux_at(const FS &fs, double g, H2 &hm, H2 &hp, double b0 = 0.0, double b1 = 0.0)
{
    const V3 Vm0 = fs.template get<DIR, 0, -1, A>(), Vm1 = fs.template get<DIR, 0, 0, A>(),
             Vm2 = fs.template get<DIR, 0, 1, A>();
    const V3 Vp0 = fs.template get<DIR, 1, -1, A>(), Vp1 = fs.template get<DIR, 1, 0, A>(),
             Vp2 = fs.template get<DIR, 1, 1, A>();
    V3 Pm0 = gauss_pt2<0>(Vm0, Vm1, Vm2), Pm1 = gauss_pt2<1>(Vm0, Vm1, Vm2);
    V3 Pp0 = gauss_pt2<0>(Vp0, Vp1, Vp2), Pp1 = gauss_pt2<1>(Vp0, Vp1, Vp2);
    hm.g[0] = Pm0.c[0]; hm.g[1] = Pm1.c[0];
    hp.g[0] = Pp0.c[0]; hp.g[1] = Pp1.c[0];
    if constexpr (FS::surf) {
        Pm0.c[0] = Pm0.c[0] - b0; Pp0.c[0] = Pp0.c[0] - b0;
        Pm1.c[0] = Pm1.c[0] - b1; Pp1.c[0] = Pp1.c[0] - b1;
    }
    const V3 F0 = llf2<DIR>(Pm0, Pp0, g);
    const V3 F1 = llf2<DIR>(Pm1, Pp1, g);
    V3 F;
#pragma unroll
    for (int c = 0; c < 3; c++) F.c[c] = 0.5 * (F0.c[c] + F1.c[c]);
    return F;
}

template <int DIR, int W, int A, class FS>
NMG2D_INL H2 face_depth_at(const FS &fs)
{
    const V3 V0 = fs.template get<DIR, W, -1, A>(), V1 = fs.template get<DIR, W, 0, A>(),
             V2 = fs.template get<DIR, W, 1, A>();
    H2 hg;
    hg.g[0] = gauss_pt2<0>(V0, V1, V2).c[0];
    hg.g[1] = gauss_pt2<1>(V0, V1, V2).c[0];
    return hg;
}

// (i, j): the row cell; h_own: its depth (perturbed when the column perturbs it), which the
// surface variant's source needs.
template <class FS>
NMG2D_INL V3 assemble_residual(const FS &fs, const Inst2D &I, const double bx[4], const double by[4], int i = 0,
                               int j = 0, double h_own = 0.0)
{
    H2 hx0, hx1, hx2, hx3, hy0, hy1, hy2, hy3, dum;
    // b at the Gauss points of the cell's four faces (surface variant)
    double bxm0 = 0.0, bxm1 = 0.0, bxp0 = 0.0, bxp1 = 0.0, bym0 = 0.0, bym1 = 0.0, byp0 = 0.0, byp1 = 0.0;
    if constexpr (FS::surf) {
        const long long fx = ((long long)j * (I.Nx + 1) + i) * 2, fy = ((long long)j * I.Nx + i) * 2;
        bxm0 = I.zfx[fx]; bxm1 = I.zfx[fx + 1]; bxp0 = I.zfx[fx + 2]; bxp1 = I.zfx[fx + 3];
        bym0 = I.zfy[fy]; bym1 = I.zfy[fy + 1];
        byp0 = I.zfy[fy + 2 * I.Nx]; byp1 = I.zfy[fy + 2 * I.Nx + 1];
    }
    const V3 fxm = face_flux_at<0, -1>(fs, I.g, dum, hx1, bxm0, bxm1);    // x_{i-1/2}: plus state from cell i
    const V3 fxp = face_flux_at<0, 0>(fs, I.g, hx2, dum, bxp0, bxp1);     // x_{i+1/2}: minus state from cell i
    const V3 fym = face_flux_at<1, -1>(fs, I.g, dum, hy1, bym0, bym1);
    const V3 fyp = face_flux_at<1, 0>(fs, I.g, hy2, dum, byp0, byp1);
    hx0 = face_depth_at<0, 1, -2>(fs);                        // x_{i-3/2}: plus state, cell i-1
    hx3 = face_depth_at<0, 0, 1>(fs);                         // x_{i+3/2}: minus state, cell i+1
    hy0 = face_depth_at<1, 1, -2>(fs);
    hy3 = face_depth_at<1, 0, 1>(fs);
    // the surface variant integrates (eta_h - eta_ij) b_x by Gauss points and the rest exactly
    double eta = 0.0;
    if constexpr (FS::surf) eta = h_own + I.zavg[((long long)j + 2) * (I.Nx + 4) + i + 2];
    // S2: the cubic in x along each y Gauss line beta at the x Gauss points gamma
    double s2 = 0.0;
#pragma unroll
    for (int be = 0; be < 2; be++) {
        const double h0 = cubic_at2<0>(hx0.g[be], hx1.g[be], hx2.g[be], hx3.g[be]);
        s2 = s2 + I.g * (FS::surf ? h0 - eta : h0) * bx[2 * be + 0];
        const double h1 = cubic_at2<1>(hx0.g[be], hx1.g[be], hx2.g[be], hx3.g[be]);
        s2 = s2 + I.g * (FS::surf ? h1 - eta : h1) * bx[2 * be + 1];
    }
    // S3: the cubic in y along each x Gauss line gamma at the y Gauss points beta
    double s3 = 0.0;
#pragma unroll
    for (int ga = 0; ga < 2; ga++) {
        const double h0 = cubic_at2<0>(hy0.g[ga], hy1.g[ga], hy2.g[ga], hy3.g[ga]);
        s3 = s3 + I.g * (FS::surf ? h0 - eta : h0) * by[0 + ga];
        const double h1 = cubic_at2<1>(hy0.g[ga], hy1.g[ga], hy2.g[ga], hy3.g[ga]);
        s3 = s3 + I.g * (FS::surf ? h1 - eta : h1) * by[2 + ga];
    }
    double S2 = -(I.dx * I.dy / 4.0) * s2;
    double S3 = -(I.dx * I.dy / 4.0) * s3;
    if constexpr (FS::surf) {
        double e2 = 0.0;
        e2 = e2 + I.g * (eta * (bxp0 - bxm0) - (bxp0 * bxp0 - bxm0 * bxm0) / 2.0);
        e2 = e2 + I.g * (eta * (bxp1 - bxm1) - (bxp1 * bxp1 - bxm1 * bxm1) / 2.0);
        double e3 = 0.0;
        e3 = e3 + I.g * (eta * (byp0 - bym0) - (byp0 * byp0 - bym0 * bym0) / 2.0);
        e3 = e3 + I.g * (eta * (byp1 - bym1) - (byp1 * byp1 - bym1 * bym1) / 2.0);
        S2 = -(I.dx * I.dy / 4.0) * s2 - (I.dy / 2.0) * e2;
        S3 = -(I.dx * I.dy / 4.0) * s3 - (I.dx / 2.0) * e3;
    }
    V3 R;
    R.c[0] = (fxp.c[0] - fxm.c[0]) / I.dx + (fyp.c[0] - fym.c[0]) / I.dy;
    R.c[1] = (fxp.c[1] - fxm.c[1]) / I.dx + (fyp.c[1] - fym.c[1]) / I.dy - S2 / (I.dx * I.dy);
    R.c[2] = (fxp.c[2] - fxm.c[2]) / I.dx + (fyp.c[2] - fym.c[2]) / I.dy - S3 / (I.dx * I.dy);
    return R;
}

// ---- ghost cells ---------------------------------------------------------------------------

// the value of side k (0 left, 1 right, 2 bottom, 3 top) out of four scalars
NMG2D_INL double side4(int k, double a0, double a1, double a2, double a3)
{
    return k == 0 ? a0 : (k == 1 ? a1 : (k == 2 ? a2 : a3));
}

// state in LDS: s[c][y][x] for cells (i0 - 2 + x, j0 - 2 + y); SURF: z[y][x], the cell averages
// of b of the same cells (ghosts included)
template <bool SURF>
struct LdsStateT {
    static constexpr bool surf = SURF;
    const double *s, *z;
    int i0, j0;
    NMG2D_INL double operator()(int c, int i, int j) const
    {
        NMG2D_CHECK(c >= 0 && c < 3 && j - j0 + 2 >= 0 && j - j0 + 2 < kSY && i - i0 + 2 >= 0 && i - i0 + 2 < kSX);
        return s[(c * kSY + (j - j0 + 2)) * kSX + (i - i0 + 2)];
    }
    NMG2D_INL double zb(int i, int j) const
    {
        NMG2D_CHECK(j - j0 + 2 >= 0 && j - j0 + 2 < kSY && i - i0 + 2 >= 0 && i - i0 + 2 < kSX);
        return z[(j - j0 + 2) * kSX + (i - i0 + 2)];
    }
};

// state in global memory [3][Ny][Nx]; SURF: zavg [Ny+4][Nx+4] (cells -2..Nx+1 x -2..Ny+1)
template <bool SURF>
struct GlobalStateT {
    static constexpr bool surf = SURF;
    const double *U, *zavg;
    int Nx, Ny;
    NMG2D_INL double operator()(int c, int i, int j) const
    {
        NMG2D_CHECK(c >= 0 && c < 3 && i >= 0 && i < Nx && j >= 0 && j < Ny);
        return U[((long long)c * Ny + j) * Nx + i];
    }
    NMG2D_INL double zb(int i, int j) const
    {
        NMG2D_CHECK(i >= -2 && i < Nx + 2 && j >= -2 && j < Ny + 2);
        return zavg[((long long)j + 2) * (Nx + 4) + i + 2];
    }
};

// Cell (i, j), ghosts included (y sides first, then x sides), with component pm of the interior
// cell (pi, pj) raised by eps; a ghost built from that cell follows it.
template <class ST>
NMG2D_INL V3 cell2(const Inst2D &I, const ST &st, int i, int j, int pi, int pj, int pm, double eps)
{
    int ii = i, jj = j, flip_u = 0, flip_v = 0, state = -1, set_h = -1, set_q = -1;
    if (j < 0 || j >= I.Ny) {
        const int side = j < 0 ? 2 : 3;
        int kind = j < 0 ? I.bc_kind[2] : I.bc_kind[3];
        if (side == 2 && I.bc_kind[2] == NMG_BC_WALL && I.wall_x > I.x0) {
            const double xc = I.x0 + (i + 0.5) * I.dx;
            kind = xc < I.wall_x ? NMG_BC_EXTRAP : NMG_BC_WALL;
        }
        const int b = j < 0 ? 0 : I.Ny - 1;
        const int m = j < 0 ? -1 - j : 2 * I.Ny - 1 - j;
        jj = b;
        if (kind == NMG_BC_WALL) { jj = m; flip_v = 1; }
        else if (kind == NMG_BC_STATE) state = side;
        else if (kind == NMG_BC_DISCHARGE) set_q = side;
        else if (kind == NMG_BC_DEPTH) set_h = side;
    }
    if (i < 0 || i >= I.Nx) {
        const int side = i < 0 ? 0 : 1;
        const int kind = i < 0 ? I.bc_kind[0] : I.bc_kind[1];
        const int b = i < 0 ? 0 : I.Nx - 1;
        const int m = i < 0 ? -1 - i : 2 * I.Nx - 1 - i;
        ii = b;
        if (kind == NMG_BC_WALL) { ii = m; flip_u = 1; }
        else if (kind == NMG_BC_STATE) state = side;
        else if (kind == NMG_BC_DISCHARGE) set_q = side;
        else if (kind == NMG_BC_DEPTH) set_h = side;
    }
    V3 out;
    if (state >= 0) {
        const double h = side4(state, I.bc_h[0], I.bc_h[1], I.bc_h[2], I.bc_h[3]);
        out.c[0] = h;
        out.c[1] = h * side4(state, I.bc_u[0], I.bc_u[1], I.bc_u[2], I.bc_u[3]);
        out.c[2] = h * side4(state, I.bc_v[0], I.bc_v[1], I.bc_v[2], I.bc_v[3]);
        return out;
    }
    const bool hit = ii == pi && jj == pj;
#pragma unroll
    for (int c = 0; c < 3; c++) {
        const double x = st(c, ii, jj);
        out.c[c] = (hit && c == pm) ? x + eps : x;
    }
    if (flip_u) out.c[1] = -out.c[1];
    if (flip_v) out.c[2] = -out.c[2];
    if constexpr (ST::surf)      // a ghost that copies a depth copies the surface
        if (ii != i || jj != j) out.c[0] = out.c[0] + st.zb(ii, jj) - st.zb(i, j);
    if (set_h >= 0) out.c[0] = side4(set_h, I.bc_h[0], I.bc_h[1], I.bc_h[2], I.bc_h[3]);
    if (set_q >= 0) {
        const double q = side4(set_q, I.bc_q[0], I.bc_q[1], I.bc_q[2], I.bc_q[3]);
        if (set_q < 2) out.c[1] = q;
        else out.c[2] = q;
    }
    return out;
}

// thread t of n stages its share of the tile's state (and, for the surface variant, the cell
// averages of b of the same cells, ghosts included, into z)
NMG2D_INL void stage_tile(const Inst2D &I, int i0, int j0, double *s, int t, int n, double *z = nullptr)
{
    for (int e = t; e < 3 * kSY * kSX; e += n) {
        const int c = e / (kSY * kSX), r = (e / kSX) % kSY, q = e % kSX;
        const int i = i0 - 2 + q, j = j0 - 2 + r;
        const bool ok = i >= 0 && i < I.Nx && j >= 0 && j < I.Ny;
        s[e] = ok ? I.U[((long long)c * I.Ny + j) * I.Nx + i] : 0.0;
    }
    if (z)
        for (int e = t; e < kSY * kSX; e += n) {
            const int r = e / kSX, q = e % kSX;
            const int i = i0 - 2 + q, j = j0 - 2 + r;
            const bool ok = i >= -2 && i < I.Nx + 2 && j >= -2 && j < I.Ny + 2;
            z[e] = ok ? I.zavg[((long long)j + 2) * (I.Nx + 4) + i + 2] : 0.0;
        }
}

// ---- residual -------------------------------------------------------------------------------

NMG2D_INL void load_slopes(const Inst2D &I, int i, int j, double bx[4], double by[4])
{
    const long long g = ((long long)j * I.Nx + i) * 4;
#pragma unroll
    for (int e = 0; e < 4; e++) {
        bx[e] = I.bx[g + e];
        by[e] = I.by[g + e];
    }
}

// ---- Jacobian -------------------------------------------------------------------------------

// Block b of the cross stencil of eq. (21): centre, x-2, x-1, x+1, x+2, y-2, y-1, y+1, y+2.
// Output: J[(b*9 + l*3 + m) * M + slot], the column (b, m) of row l, in the cell order Pm.
struct JacOut {
    long long M, slot;
    double R0, R1, R2, rn, alpha, eps;
};

template <typename T>
NMG2D_INL void store_column(T *J, const JacOut &o, int b, int m, const V3 &Rp, double d[3])
{
    double c0 = (Rp.c[0] - o.R0) / o.eps;
    double c1 = (Rp.c[1] - o.R1) / o.eps;
    double c2 = (Rp.c[2] - o.R2) / o.eps;
    if (b == 0) {
        if (m == 0) c0 += o.alpha * o.rn;
        else if (m == 1) c1 += o.alpha * o.rn;
        else c2 += o.alpha * o.rn;
    }
    J[(b * 9 + 0 * 3 + m) * o.M + o.slot] = (T)c0;
    J[(b * 9 + 1 * 3 + m) * o.M + o.slot] = (T)c1;
    J[(b * 9 + 2 * 3 + m) * o.M + o.slot] = (T)c2;
    d[0] = c0; d[1] = c1; d[2] = c2;
}

template <typename T>
NMG2D_INL void store_zero_column(T *J, const JacOut &o, int b, int m)
{
#pragma unroll
    for (int l = 0; l < 3; l++) J[(b * 9 + l * 3 + m) * o.M + o.slot] = (T)0.0;
}

// inverse of the diagonal block D (row-major d[l*3+m]) by the adjugate over the determinant
template <typename T>
NMG2D_INL void store_dinv(T *Dinv, long long M, long long slot, const double D[9])
{
    const double c00 = D[4] * D[8] - D[5] * D[7];
    const double c01 = D[5] * D[6] - D[3] * D[8];
    const double c02 = D[3] * D[7] - D[4] * D[6];
    const double det = D[0] * c00 + D[1] * c01 + D[2] * c02;
    Dinv[0 * M + slot] = (T)(c00 / det);
    Dinv[1 * M + slot] = (T)((D[2] * D[7] - D[1] * D[8]) / det);
    Dinv[2 * M + slot] = (T)((D[1] * D[5] - D[2] * D[4]) / det);
    Dinv[3 * M + slot] = (T)(c01 / det);
    Dinv[4 * M + slot] = (T)((D[0] * D[8] - D[2] * D[6]) / det);
    Dinv[5 * M + slot] = (T)((D[2] * D[3] - D[0] * D[5]) / det);
    Dinv[6 * M + slot] = (T)(c02 / det);
    Dinv[7 * M + slot] = (T)((D[1] * D[6] - D[0] * D[7]) / det);
    Dinv[8 * M + slot] = (T)((D[0] * D[4] - D[1] * D[3]) / det);
}

// a row whose residual involves a ghost cell: within two cells of a side
NMG2D_INL bool border_row(const Inst2D &I, int i, int j)
{
    return i < 2 || j < 2 || i >= I.Nx - 2 || j >= I.Ny - 2;
}

// Tables of the interior kernel for a tile of TX x TY cells: the face states its rows use, three
// components in line order (depth, momentum along the line, momentum across it).  Set p = 0, 1, 2:
// the state with one component of the p-th of its three cells raised by eps; set 3: unperturbed.
template <int TX, int TY>
struct JacTile {
    static constexpr int SX = TX + 4, SY = TY + 4;                 // staged state (halo 2)
    static constexpr int XA = TX + 3, XL = TY + 2, YA = TY + 3, YL = TX + 2;
    static constexpr int XS = 6 * XL * XA, SET = XS + 6 * YL * YA;
    static constexpr int STATES = 2 * XL * (XA - 1);               // x (and, by symmetry of the count, y) states
    static_assert(XL * (XA - 1) == YL * (YA - 1), "as many y states as x states");
    // component 0 of the state of side W of face A on line K, relative to the row cell's base
    template <int DIR, int W, int K, int A>
    static constexpr int at() { return DIR == 0 ? (W * XL + 1 + K) * XA + 2 + A : XS + (W * YL + 1 + K) * YA + 2 + A; }
    template <int DIR>
    static constexpr int comp() { return DIR == 0 ? 2 * XL * XA : 2 * YL * YA; }
};

// A column's perturbed cell as direction DIR sees it: d along the line, k the line.  The state of side
// W of face A on line K uses the cells A - 1 + W .. A + 1 + W of its line.
struct Hit {
    int d, k;
    template <int W, int K, int A>
    NMG2D_INL int set() const
    {
        const int p = d - (A - 1 + W);
        return K == k && p >= 0 && p <= 2 ? p : 3;
    }
    // one of the states that the flux through face A, or the depth of side W there, is formed from
    template <int A>
    NMG2D_INL bool flux() const { return k >= -1 && k <= 1 && d >= A - 1 && d <= A + 2; }
    template <int W, int A>
    NMG2D_INL bool depth() const { return k >= -1 && k <= 1 && d >= A - 1 + W && d <= A + 1 + W; }
};

// tables of the unperturbed states alone
struct NoHit {
    template <int W, int K, int A>
    NMG2D_INL int set() const { return 0; }
};

template <class TL, int DIR, int W, int K, int A, class H>
NMG2D_INL V3 tab_state(const double *tab, const H &h)
{
    const double *q = tab + h.template set<W, K, A>() * TL::SET + TL::template at<DIR, W, K, A>();
    return V3{{q[0], q[TL::template comp<DIR>()], q[2 * TL::template comp<DIR>()]}};
}

// flux through face A in direction DIR, line order; hm, hp and b0, b1 as in face_flux_at
template <class TL, int DIR, int A, bool SURF, class H>
NMG2D_INL V3 tab_flux(const double *tab, const H &h, double g, H2 &hm, H2 &hp, double b0, double b1)
{
    const V3 Vm0 = tab_state<TL, DIR, 0, -1, A>(tab, h), Vm1 = tab_state<TL, DIR, 0, 0, A>(tab, h),
             Vm2 = tab_state<TL, DIR, 0, 1, A>(tab, h);
    const V3 Vp0 = tab_state<TL, DIR, 1, -1, A>(tab, h), Vp1 = tab_state<TL, DIR, 1, 0, A>(tab, h),
             Vp2 = tab_state<TL, DIR, 1, 1, A>(tab, h);
    V3 Pm0 = gauss_pt2<0>(Vm0, Vm1, Vm2), Pm1 = gauss_pt2<1>(Vm0, Vm1, Vm2);
    V3 Pp0 = gauss_pt2<0>(Vp0, Vp1, Vp2), Pp1 = gauss_pt2<1>(Vp0, Vp1, Vp2);
    hm.g[0] = Pm0.c[0]; hm.g[1] = Pm1.c[0];
    hp.g[0] = Pp0.c[0]; hp.g[1] = Pp1.c[0];
    if constexpr (SURF) {
        Pm0.c[0] = Pm0.c[0] - b0; Pp0.c[0] = Pp0.c[0] - b0;
        Pm1.c[0] = Pm1.c[0] - b1; Pp1.c[0] = Pp1.c[0] - b1;
    }
    const V3 F0 = llf2<0>(Pm0, Pp0, g), F1 = llf2<0>(Pm1, Pp1, g);
    V3 F;
#pragma unroll
    for (int c = 0; c < 3; c++) F.c[c] = 0.5 * (F0.c[c] + F1.c[c]);
    return F;
}

template <class TL, int DIR, int W, int A, class H>
NMG2D_INL H2 tab_depth(const double *tab, const H &h)
{
    const V3 V0 = tab_state<TL, DIR, W, -1, A>(tab, h), V1 = tab_state<TL, DIR, W, 0, A>(tab, h),
             V2 = tab_state<TL, DIR, W, 1, A>(tab, h);
    return H2{{gauss_pt2<0>(V0, V1, V2).c[0], gauss_pt2<1>(V0, V1, V2).c[0]}};
}

// What the residual of a row is assembled from: the fluxes through its four faces (line order) and, per
// direction, the depths of its lines' cubics at x - 3/2, - 1/2, + 1/2, + 3/2
struct RowParts {
    V3 fxm, fxp, fym, fyp;
    H2 hx[4], hy[4];
};

// the parts a perturbed cell reaches, the others from `o`
template <class TL, bool SURF>
NMG2D_INL void row_parts(RowParts &r, const RowParts &o, const double *tx, const double *ty, const Hit &hx, const Hit &hy,
                         double g, const double zx[4], const double zy[4])
{
    H2 dum;
    r = o;
    if (hx.flux<-1>()) r.fxm = tab_flux<TL, 0, -1, SURF>(tx, hx, g, dum, r.hx[1], zx[0], zx[1]);
    if (hx.flux<0>()) r.fxp = tab_flux<TL, 0, 0, SURF>(tx, hx, g, r.hx[2], dum, zx[2], zx[3]);
    if (hy.flux<-1>()) r.fym = tab_flux<TL, 1, -1, SURF>(ty, hy, g, dum, r.hy[1], zy[0], zy[1]);
    if (hy.flux<0>()) r.fyp = tab_flux<TL, 1, 0, SURF>(ty, hy, g, r.hy[2], dum, zy[2], zy[3]);
    if (hx.depth<1, -2>()) r.hx[0] = tab_depth<TL, 0, 1, -2>(tx, hx);
    if (hx.depth<0, 1>()) r.hx[3] = tab_depth<TL, 0, 0, 1>(tx, hx);
    if (hy.depth<1, -2>()) r.hy[0] = tab_depth<TL, 1, 1, -2>(ty, hy);
    if (hy.depth<0, 1>()) r.hy[3] = tab_depth<TL, 1, 0, 1>(ty, hy);
}

// R_ij from its parts: the operations of assemble_residual.  zx, zy: b at the Gauss points of the
// cell's faces (lower face, then upper; surface variant), eta: the cell's surface there.
template <bool SURF>
NMG2D_INL V3 row_residual(const RowParts &r, const Inst2D &I, const Recip &rdx, const Recip &rdy, const Recip &rdd,
                          const double bx[4], const double by[4], const double zx[4], const double zy[4], double eta)
{
    double s2 = 0.0, s3 = 0.0;
#pragma unroll
    for (int be = 0; be < 2; be++) {
        const double h0 = cubic_at2<0>(r.hx[0].g[be], r.hx[1].g[be], r.hx[2].g[be], r.hx[3].g[be]);
        s2 = s2 + I.g * (SURF ? h0 - eta : h0) * bx[2 * be + 0];
        const double h1 = cubic_at2<1>(r.hx[0].g[be], r.hx[1].g[be], r.hx[2].g[be], r.hx[3].g[be]);
        s2 = s2 + I.g * (SURF ? h1 - eta : h1) * bx[2 * be + 1];
    }
#pragma unroll
    for (int ga = 0; ga < 2; ga++) {
        const double h0 = cubic_at2<0>(r.hy[0].g[ga], r.hy[1].g[ga], r.hy[2].g[ga], r.hy[3].g[ga]);
        s3 = s3 + I.g * (SURF ? h0 - eta : h0) * by[0 + ga];
        const double h1 = cubic_at2<1>(r.hy[0].g[ga], r.hy[1].g[ga], r.hy[2].g[ga], r.hy[3].g[ga]);
        s3 = s3 + I.g * (SURF ? h1 - eta : h1) * by[2 + ga];
    }
    double S2 = -(I.dx * I.dy / 4.0) * s2;
    double S3 = -(I.dx * I.dy / 4.0) * s3;
    if constexpr (SURF) {
        double e2 = 0.0, e3 = 0.0;
#pragma unroll
        for (int q = 0; q < 2; q++) {
            e2 = e2 + I.g * (eta * (zx[2 + q] - zx[q]) - (zx[2 + q] * zx[2 + q] - zx[q] * zx[q]) / 2.0);
            e3 = e3 + I.g * (eta * (zy[2 + q] - zy[q]) - (zy[2 + q] * zy[2 + q] - zy[q] * zy[q]) / 2.0);
        }
        S2 = -(I.dx * I.dy / 4.0) * s2 - (I.dy / 2.0) * e2;
        S3 = -(I.dx * I.dy / 4.0) * s3 - (I.dx / 2.0) * e3;
    }
    V3 R;
    R.c[0] = rdx.of(r.fxp.c[0] - r.fxm.c[0]) + rdy.of(r.fyp.c[0] - r.fym.c[0]);
    R.c[1] = rdx.of(r.fxp.c[1] - r.fxm.c[1]) + rdy.of(r.fyp.c[2] - r.fym.c[2]) - rdd.of(S2);
    R.c[2] = rdx.of(r.fxp.c[2] - r.fxm.c[2]) + rdy.of(r.fyp.c[1] - r.fym.c[1]) - rdd.of(S3);
    return R;
}

// The blocks that column group `group` of `groups` forms (bit b: block b): blocks go, the costly ones
// (whose cell reaches all four faces: the centre and the cells next to it, diagonals included) first, to
// the group with the least work so far
constexpr unsigned column_group(int nb, int groups, int group)
{
    unsigned mask[8] = {};
    int load[8] = {};
    for (int pass = 0; pass < 2; pass++)
        for (int b = 0; b < nb; b++) {
            const int dx = stencil_dx(21, b), dy = stencil_dy(21, b);
            const bool near = dx >= -1 && dx <= 1 && dy >= -1 && dy <= 1;
            if (near != (pass == 0)) continue;
            int best = 0;
            for (int q = 1; q < groups; q++)
                if (load[q] < load[best]) best = q;
            mask[best] |= 1u << b;
            load[best] += near ? 5 : 2;
        }
    return mask[group];
}

// Finite-difference Jacobian (eq. 12, 13) of the rows at least two cells inside the grid (no ghost in
// their residual).  A perturbed face state serves up to five rows, so the tile forms each once per
// component (3 cells x 3 components x 4 states a cell, where every row for itself re-evaluates 60 a
// component) and the rows assemble their columns from the tables, re-forming only the fluxes
// that the perturbed cell reaches.  What bounds it is FP64 arithmetic (divisions and square roots) at
// two wavefronts per SIMD, which the tables' LDS allows: one workgroup of 512 threads per compute unit.
// The columns of a row are shared by CG = 512 / (TX TY) threads (wavefronts of their own, so the column
// is uniform): 2 on the 32 x 8 tile, 8 on the 8 x 8 tile for grids too small to fill the chip with
// the larger one.
// 1024 x 512, J9: 2050 us with every row re-evaluating its states, 1250 with cheaper divisions, 832 so;
// 64 x 32: 226, 150, 35.
constexpr int kJacNT = 512;

template <int TX, int TY>
constexpr int kJacLds = 4 * JacTile<TX, TY>::SET + 4 * JacTile<TX, TY>::SX * JacTile<TX, TY>::SY;

template <typename T, int NB, bool SURF, int TX, int TY>
__device__ __forceinline__ void interior_rows(const Inst2D &I, const Perm2D &Pm, T *J, T *rhs, T *Dinv, int i0, int j0,
                                              double *lds)
{
    typedef JacTile<TX, TY> TL;
    constexpr int CG = kJacNT / (TX * TY), SX = TL::SX, SY = TL::SY;
    static_assert(TX * TY % 64 == 0 && CG <= 8, "a wavefront forms one column at a time");
    double *const tab = lds, *const s = lds + 4 * TL::SET, *const zs = s + 3 * SY * SX;
    const int t = threadIdx.x;
    for (int e = t; e < 3 * SY * SX; e += kJacNT) {
        const int c = e / (SY * SX), r = (e / SX) % SY, q = e % SX;
        const int i = i0 - 2 + q, j = j0 - 2 + r;
        const bool ok = i >= 0 && i < I.Nx && j >= 0 && j < I.Ny;
        s[e] = ok ? I.U[((long long)c * I.Ny + j) * I.Nx + i] : 0.0;
    }
    if constexpr (SURF)
        for (int e = t; e < SY * SX; e += kJacNT) {
            const int i = i0 - 2 + e % SX, j = j0 - 2 + e / SX;
            const bool ok = i >= -2 && i < I.Nx + 2 && j >= -2 && j < I.Ny + 2;
            zs[e] = ok ? I.zavg[((long long)j + 2) * (I.Nx + 4) + i + 2] : 0.0;
        }
    __syncthreads();

    const int cell = t % (TX * TY), xi = cell % TX, xj = cell / TX;
    const int group = __builtin_amdgcn_readfirstlane(t / (TX * TY));
    const int i = i0 + xi, j = j0 + xj;
    const bool row = i < I.Nx && j < I.Ny && !border_row(I, i, j);
    const double *tx = tab + xj * TL::XA + xi, *ty = tab + xi * TL::YA + xj;
    unsigned blocks = 0;
#pragma unroll
    for (int q = 0; q < CG; q++)
        if (group == q) blocks = column_group(NB, CG, q);
    const Recip rdx(I.dx), rdy(I.dy), rdd(I.dx * I.dy);
    JacOut o;
    RowParts base;
    double bx[4], by[4], zx[4], zy[4], D[9], zc = 0.0;
    if (row) {
        const long long n = (long long)I.Nx * I.Ny, cidx = (long long)j * I.Nx + i;
        o.M = Pm.M;
        o.slot = perm2d_rows(Pm, i, j);
        o.R0 = I.R[cidx];
        o.R1 = I.R[n + cidx];
        o.R2 = I.R[2 * n + cidx];
        o.rn = I.rn[cidx];
        o.alpha = I.alpha;
        o.eps = I.eps;
        if (rhs && group == 0) {
            rhs[o.slot] = (T)o.R0;
            rhs[o.M + o.slot] = (T)o.R1;
            rhs[2 * o.M + o.slot] = (T)o.R2;
        }
        load_slopes(I, i, j, bx, by);
        if constexpr (SURF) {
            const long long fx = ((long long)j * (I.Nx + 1) + i) * 2, fy = ((long long)j * I.Nx + i) * 2;
#pragma unroll
            for (int q = 0; q < 2; q++) {
                zx[q] = I.zfx[fx + q];
                zx[2 + q] = I.zfx[fx + 2 + q];
                zy[q] = I.zfy[fy + q];
                zy[2 + q] = I.zfy[fy + 2 * I.Nx + q];
            }
            zc = zs[(xj + 2) * SX + xi + 2];
        }
    }
#pragma unroll
    for (int e = 0; e < 9; e++) D[e] = 0.0;

#pragma unroll 1
    for (int m = 0; m < 3; m++) {
        // the tables of component m (with m = 0 also the unperturbed ones): states whose cells leave the
        // grid belong to no interior row
        for (int e = t; e < (m == 0 ? 4 : 3) * 2 * TL::STATES; e += kJacNT) {
            const int p = e / (2 * TL::STATES), r = e - p * (2 * TL::STATES), dir = r / TL::STATES;
            const int q = r - dir * TL::STATES, W = q / (TL::STATES / 2), f = q - W * (TL::STATES / 2);
            const int per = dir ? TL::YA - 1 : TL::XA - 1, line = f / per, a = f - line * per + (W ? 0 : 1);
            const int t0 = (dir ? j0 : i0) - 3 + a + W, k = (dir ? i0 : j0) - 1 + line;
            if (t0 < 0 || t0 + 2 >= (dir ? I.Ny : I.Nx) || k < 0 || k >= (dir ? I.Nx : I.Ny)) continue;
            const int c0 = dir ? (a + W - 1) * SX + line + 1 : (line + 1) * SX + a + W - 1, step = dir ? SX : 1;
            V3 S[3];
            double z[3] = {0.0, 0.0, 0.0};
#pragma unroll
            for (int x = 0; x < 3; x++) {
                const double *v = s + c0 + x * step;
                double h = v[0], hu = v[SY * SX], hv = v[2 * SY * SX];
                if (x == p) {
                    h = m == 0 ? h + I.eps : h;
                    hu = m == 1 ? hu + I.eps : hu;
                    hv = m == 2 ? hv + I.eps : hv;
                }
                S[x] = dir ? V3{{h, hv, hu}} : V3{{h, hu, hv}};
                if constexpr (SURF) z[x] = zs[c0 + x * step];
            }
            const V3 v = W ? face_state_line<SURF>(S[2], S[1], S[0], I.g, z[2], z[1], z[0])
                           : face_state_line<SURF>(S[0], S[1], S[2], I.g, z[0], z[1], z[2]);
            double *w = tab + p * TL::SET + (dir ? TL::XS + (W * TL::YL + line) * TL::YA : (W * TL::XL + line) * TL::XA) + a;
            const int comp = dir ? TL::template comp<1>() : TL::template comp<0>();
#pragma unroll
            for (int c = 0; c < 3; c++) w[c * comp] = v.c[c];
        }
        __syncthreads();
        if (row) {
            if (m == 0) {
                const Hit none{100, 0};
                H2 dum;
                base.fxm = tab_flux<TL, 0, -1, SURF>(tx, none, I.g, dum, base.hx[1], zx[0], zx[1]);
                base.fxp = tab_flux<TL, 0, 0, SURF>(tx, none, I.g, base.hx[2], dum, zx[2], zx[3]);
                base.fym = tab_flux<TL, 1, -1, SURF>(ty, none, I.g, dum, base.hy[1], zy[0], zy[1]);
                base.fyp = tab_flux<TL, 1, 0, SURF>(ty, none, I.g, base.hy[2], dum, zy[2], zy[3]);
                base.hx[0] = tab_depth<TL, 0, 1, -2>(tx, none);
                base.hx[3] = tab_depth<TL, 0, 0, 1>(tx, none);
                base.hy[0] = tab_depth<TL, 1, 1, -2>(ty, none);
                base.hy[3] = tab_depth<TL, 1, 0, 1>(ty, none);
            }
#pragma unroll 1
            for (int b = 0; b < NB; b++) {
                if (!(blocks >> b & 1)) continue;
                const int dx = stencil_dx(21, b), dy = stencil_dy(21, b);
                RowParts r;
                row_parts<TL, SURF>(r, base, tx, ty, Hit{dx, dy}, Hit{dy, dx}, I.g, zx, zy);
                double eta = 0.0;
                if constexpr (SURF) {
                    const double x = s[(xj + 2) * SX + xi + 2];
                    eta = (b == 0 && m == 0 ? x + I.eps : x) + zc;
                }
                const V3 Rp = row_residual<SURF>(r, I, rdx, rdy, rdd, bx, by, zx, zy, eta);
                double d[3];
                store_column(J, o, b, m, Rp, d);
                if (b == 0) {
#pragma unroll
                    for (int l = 0; l < 3; l++)
#pragma unroll
                        for (int c = 0; c < 3; c++)
                            if (c == m) D[l * 3 + c] = d[l];
                }
            }
        }
        __syncthreads();
    }
    if (row && Dinv && (blocks & 1)) store_dinv(Dinv, o.M, o.slot, D);
}

template <typename T, int NB, bool SURF, int TX, int TY>
__global__ void __launch_bounds__(kJacNT) k_jacobian2d(Inst2D I, Perm2D Pm, T *J, T *rhs, T *Dinv)
{
    __shared__ double lds[kJacLds<TX, TY>];
    interior_rows<T, NB, SURF, TX, TY>(I, Pm, J, rhs, Dinv, blockIdx.x * TX, blockIdx.y * TY, lds);
}

// Face states of one column of a border row: the state of slot q at slots[(q*3 + c) * kBorderNT + lane]
// where the perturbed cell reaches it (bit q of hits), else the row's unperturbed one at base[q*3 + c].
template <bool SURF>
struct SlotFS {
    static constexpr bool surf = SURF;
    const double *slots, *base;
    unsigned long long hits;
    int lane;
    // slot of a face state: per direction 18, in the order A = -1 (6: W, K), A = 0 (6),
    // A = -2 (3: K, plus side), A = 1 (3: K, minus side)
    template <int DIR, int W, int K, int A>
    static constexpr int slot()
    {
        return DIR * 18 + (A == -1 ? (W * 3 + K + 1) : A == 0 ? 6 + W * 3 + K + 1 : A == -2 ? 12 + K + 1 : 15 + K + 1);
    }
    template <int DIR, int W, int K, int A>
    NMG2D_INL V3 get() const
    {
        constexpr int q = slot<DIR, W, K, A>();
        const bool hit = hits >> q & 1;
        V3 v;
#pragma unroll
        for (int c = 0; c < 3; c++) v.c[c] = hit ? slots[(q * 3 + c) * kBorderNT + lane] : base[q * 3 + c];
        return v;
    }
};

// slot q of the row (i, j): its direction, side, first cell along the line and line (runtime decode)
struct SlotAt {
    int dir, w, t0, k;
    SlotAt() = default;
    NMG2D_INL SlotAt(int q, int i, int j)
    {
        dir = q / 18;
        const int r = q - 18 * dir;
        int K, A;
        if (r < 6) { A = -1; w = r / 3; K = r % 3 - 1; }
        else if (r < 12) { A = 0; w = (r - 6) / 3; K = (r - 6) % 3 - 1; }
        else if (r < 15) { A = -2; w = 1; K = r - 13; }
        else { A = 1; w = 0; K = r - 16; }
        t0 = (dir ? j : i) + A - 1 + w;
        k = (dir ? i : j) + K;
    }
};

// the face state at a slot under the perturbation (pi, pj, pm), ghosts applied
template <class ST>
NMG2D_INL V3 slot_state(const Inst2D &I, const ST &st, const SlotAt &a, int pi, int pj, int pm, double eps)
{
    V3 S[3];
    double z[3] = {0.0, 0.0, 0.0};
#pragma unroll
    for (int q = 0; q < 3; q++) {
        const int t = a.t0 + (a.w ? 2 - q : q), i = a.dir ? a.k : t, j = a.dir ? t : a.k;
        const V3 U = cell2(I, st, i, j, pi, pj, pm, eps);
        S[q] = a.dir ? V3{{U.c[0], U.c[2], U.c[1]}} : U;
        if constexpr (ST::surf) z[q] = st.zb(i, j);
    }
    const V3 v = face_state_line<ST::surf>(S[0], S[1], S[2], I.g, z[0], z[1], z[2]);
    return a.dir ? V3{{v.c[0], v.c[2], v.c[1]}} : v;
}

// whether cell (i, j), ghosts included, takes its values from the cell (pi, pj) of the grid
NMG2D_INL bool follows(const Inst2D &I, int i, int j, int pi, int pj)
{
    int ii = i, jj = j;
    bool state = false;
    if (j < 0 || j >= I.Ny) {
        int kind = j < 0 ? I.bc_kind[2] : I.bc_kind[3];
        if (j < 0 && kind == NMG_BC_WALL && I.wall_x > I.x0) {
            const double xc = I.x0 + (i + 0.5) * I.dx;
            kind = xc < I.wall_x ? NMG_BC_EXTRAP : NMG_BC_WALL;
        }
        if (kind == NMG_BC_WALL) jj = j < 0 ? -1 - j : 2 * I.Ny - 1 - j;
        else jj = j < 0 ? 0 : I.Ny - 1;
        if (kind == NMG_BC_STATE) state = true;
    }
    if (i < 0 || i >= I.Nx) {
        const int kind = i < 0 ? I.bc_kind[0] : I.bc_kind[1];
        if (kind == NMG_BC_WALL) ii = i < 0 ? -1 - i : 2 * I.Nx - 1 - i;
        else ii = i < 0 ? 0 : I.Nx - 1;
        if (kind == NMG_BC_STATE) state = true;
    }
    return !state && ii == pi && jj == pj;
}

NMG2D_INL bool slot_follows(const Inst2D &I, const SlotAt &a, int pi, int pj)
{
    bool hit = false;
#pragma unroll
    for (int q = 0; q < 3; q++) {
        const int t = a.t0 + q;
        hit = hit || follows(I, a.dir ? a.k : t, a.dir ? t : a.k, pi, pj);
    }
    return hit;
}

// the cell of border row number r (rows within two cells of a side, bottom band, top band, then
// the two side bands of the rows in between)
NMG2D_INL void border_cell(const Inst2D &I, long long r, int &i, int &j)
{
    const int nb = I.Ny < 2 ? I.Ny : 2;                 // bottom band rows
    const int jt = I.Ny - 2 > nb ? I.Ny - 2 : nb;       // first top band row
    const long long bottom = (long long)nb * I.Nx, top = (long long)(I.Ny - jt) * I.Nx;
    if (r < bottom) { j = (int)(r / I.Nx); i = (int)(r - (long long)j * I.Nx); return; }
    r -= bottom;
    if (r < top) { j = jt + (int)(r / I.Nx); i = (int)(r - (long long)(j - jt) * I.Nx); return; }
    r -= top;
    const int side = I.Nx < 4 ? I.Nx : 4;                // side cells per middle row
    j = nb + (int)(r / side);
    const int k = (int)(r - (long long)(j - nb) * side);
    i = (I.Nx <= 4 || k < 2) ? k : I.Nx - 4 + k;
}

long long border_rows2d(int Nx, int Ny)
{
    const long long inner = (long long)(Nx > 4 ? Nx - 4 : 0) * (Ny > 4 ? Ny - 4 : 0);
    return (long long)Nx * Ny - inner;
}

// Jacobian of the border rows, from the state in global memory.  A workgroup of 256 threads takes
// kBorderNT / LPR rows: it forms their 36 unperturbed states, lists the (row, block, state) triples
// whose state follows the perturbed cell (through a ghost or directly; about 7 of 36 per column),
// forms those for the three components, and then assembles a column per thread.  Bound by the chain
// of one state after another (every column's 36 in one thread: 81 us at 64 x 32, 470 us at
// 1024 x 512; the list spread over the threads: 20 and 115 us).  A row takes LPR lanes of a wavefront
// (32 for the 27 columns of J9, 64 for the 63 of J21), so the lanes of its three diagonal-block columns
// can hand their FP64 values to the row's first lane, which writes the inverse of the diagonal block.
constexpr int kBorderThreads = 256;

template <int NB>
struct BorderLds {
    static constexpr int LPR = NB == 9 ? 32 : 64, RPW = kBorderNT / LPR;
    double slots[kSlots * 3 * kBorderNT];
    double base[RPW * kSlots * 3];
    unsigned long long hits[RPW * NB];
    unsigned short list[RPW * NB * kSlots];
    int count;
};

template <typename T, int NB, bool SURF, int NT>
__device__ __forceinline__ void border_rows(const Inst2D &I, const Perm2D &Pm, T *J, T *rhs, T *Dinv, long long r0,
                                            long long nrows, BorderLds<NB> &B)
{
    constexpr int LPR = BorderLds<NB>::LPR, RPW = BorderLds<NB>::RPW;
    static_assert(kBorderNT % LPR == 0 && NT >= kBorderNT, "a workgroup holds whole rows");
    double *const slots = B.slots, *const base = B.base;
    unsigned long long *const hits = B.hits;
    unsigned short *const list = B.list;
    int &count = B.count;
    const int t = threadIdx.x;
    const GlobalStateT<SURF> st{I.U, I.zavg, I.Nx, I.Ny};
    for (int e = t; e < RPW * NB; e += NT) hits[e] = 0;
    if (t == 0) count = 0;
    __syncthreads();
    for (int e = t; e < RPW * kSlots; e += NT) {
        const int row = e / kSlots, q = e - row * kSlots;
        if (r0 + row >= nrows) continue;
        int i, j;
        border_cell(I, r0 + row, i, j);
        const V3 v = slot_state(I, st, SlotAt(q, i, j), -1000, -1000, 0, 0.0);
#pragma unroll
        for (int c = 0; c < 3; c++) base[(row * kSlots + q) * 3 + c] = v.c[c];
    }
    for (int e = t; e < RPW * NB * kSlots; e += NT) {
        const int rb = e / kSlots, q = e - rb * kSlots, row = rb / NB, b = rb - row * NB;
        if (r0 + row >= nrows) continue;
        int i, j;
        border_cell(I, r0 + row, i, j);
        const int pi = i + stencil_dx(21, b), pj = j + stencil_dy(21, b);
        if (pi < 0 || pi >= I.Nx || pj < 0 || pj >= I.Ny || !slot_follows(I, SlotAt(q, i, j), pi, pj)) continue;
        atomicOr(&hits[rb], 1ULL << q);
        list[atomicAdd(&count, 1)] = (unsigned short)e;      // in any order: the states are independent
    }
    __syncthreads();
    for (int e = t; e < 3 * count; e += NT) {
        const int m = e % 3, x = list[e / 3], rb = x / kSlots, q = x - rb * kSlots, row = rb / NB, b = rb - row * NB;
        int i, j;
        border_cell(I, r0 + row, i, j);
        const V3 v = slot_state(I, st, SlotAt(q, i, j), i + stencil_dx(21, b), j + stencil_dy(21, b), m, I.eps);
#pragma unroll
        for (int c = 0; c < 3; c++) slots[(q * 3 + c) * kBorderNT + row * LPR + b * 3 + m] = v.c[c];
    }
    __syncthreads();
    if (t >= kBorderNT) return;
    const int row = t / LPR, col = t % LPR, b = col / 3, m = col - 3 * b;
    const bool active = r0 + row < nrows && col < 3 * NB;
    double d[3] = {0.0, 0.0, 0.0};
    long long slot = 0;
    if (active) {
        int i, j;
        border_cell(I, r0 + row, i, j);
        const long long n = (long long)I.Nx * I.Ny, cidx = (long long)j * I.Nx + i;
        JacOut o;
        o.M = Pm.M;
        o.slot = slot = perm2d_rows(Pm, i, j);
        o.R0 = I.R[cidx];
        o.R1 = I.R[n + cidx];
        o.R2 = I.R[2 * n + cidx];
        o.rn = I.rn[cidx];
        o.alpha = I.alpha;
        o.eps = I.eps;
        if (rhs && col == 0) {
            rhs[o.slot] = (T)o.R0;
            rhs[o.M + o.slot] = (T)o.R1;
            rhs[2 * o.M + o.slot] = (T)o.R2;
        }
        const int pi = i + stencil_dx(21, b), pj = j + stencil_dy(21, b);
        if (pi < 0 || pi >= I.Nx || pj < 0 || pj >= I.Ny) {
            store_zero_column(J, o, b, m);
        } else {
            double bx[4], by[4];
            load_slopes(I, i, j, bx, by);
            const SlotFS<SURF> fs{slots, base + row * kSlots * 3, hits[row * NB + b], t};
            double h_own = 0.0;
            if constexpr (SURF) {
                const double x = st(0, i, j);
                h_own = (pi == i && pj == j && m == 0) ? x + I.eps : x;
            }
            const V3 Rp = assemble_residual(fs, I, bx, by, i, j, h_own);
            store_column(J, o, b, m, Rp, d);
        }
    }
    if (!Dinv) return;   // uniform over the launch
    // the diagonal block's columns m = 0, 1, 2 sit in lanes 0, 1, 2 of the row's LPR
    const int first = t & ~(LPR - 1);
    double D[9];
#pragma unroll
    for (int mm = 0; mm < 3; mm++)
#pragma unroll
        for (int l = 0; l < 3; l++) D[l * 3 + mm] = __shfl(d[l], first + mm, 64);
    if (active && col == 0) store_dinv(Dinv, Pm.M, slot, D);
}

template <typename T, int NB, bool SURF>
__global__ void __launch_bounds__(kBorderThreads) k_jacobian2d_border(Inst2D I, Perm2D Pm, T *J, T *rhs, T *Dinv,
                                                                      long long nrows)
{
    __shared__ BorderLds<NB> B;
    border_rows<T, NB, SURF, kBorderThreads>(I, Pm, J, rhs, Dinv, blockIdx.x * (long long)BorderLds<NB>::RPW, nrows, B);
}

// The whole Jacobian of a grid too small to fill the chip, in one launch: the interior rows' 8 x 8 tiles
// in the first workgroups, the border rows in the others, side by side (64 x 32: 55 us one after the
// other, 35 so).
template <typename T, int NB, bool SURF>
__global__ void __launch_bounds__(kJacNT) k_jacobian2d_small(Inst2D I, Perm2D Pm, T *J, T *rhs, T *Dinv, int gx, int ntiles,
                                                             long long nrows)
{
    __shared__ union Lds {
        double d[kJacLds<8, 8>];
        BorderLds<NB> b;
    } lds;
    const int g = blockIdx.x;
    if (g < ntiles) interior_rows<T, NB, SURF, 8, 8>(I, Pm, J, rhs, Dinv, g % gx * 8, g / gx * 8, lds.d);
    else border_rows<T, NB, SURF, kJacNT>(I, Pm, J, rhs, Dinv, (g - ntiles) * (long long)BorderLds<NB>::RPW, nrows, lds.b);
}

// ---- residual with each face's flux formed once ---------------------------------------------
// The face states of a tile are spread over the workgroup's threads, then the faces: a flux serves the
// cells on both sides of its face.  The tile's sum is that of four wavefronts of 64 cells.  NT = 1024
// for a grid too small to fill the chip, which waits for the chain in one thread (64 x 32: 23.5 us
// with a cell a thread, 12.5 so); 512 otherwise, two workgroups a compute unit (1024 x 512: 83 us with a
// cell a thread that forms its four fluxes itself, 69 so).
template <bool SURF, int NT>
__global__ void __launch_bounds__(NT) k_residual2d(Inst2D I, double *partial)
{
    typedef JacTile<kTX, kTY> TL;
    constexpr int CELLS = kTX * kTY, NW = CELLS / 64;
    constexpr int FX = (kTX + 1) * kTY, FY = kTX * (kTY + 1);    // faces of the tile's cells
    __shared__ double s[3 * kSY * kSX];
    __shared__ double zs[SURF ? kSY * kSX : 1];
    __shared__ double tab[TL::SET];
    __shared__ double part[7][FX + FY];        // per face: its flux, the depths on its lower and upper side
    __shared__ double red[NW];
    const int i0 = blockIdx.x * kTX, j0 = blockIdx.y * kTY, t = threadIdx.x;
    stage_tile(I, i0, j0, s, t, NT, SURF ? zs : nullptr);
    __syncthreads();
    const LdsStateT<SURF> st{s, zs, i0, j0};
    for (int e = t; e < 2 * TL::STATES; e += NT) {
        const int dir = e / TL::STATES, q = e - dir * TL::STATES, W = q / (TL::STATES / 2), f = q - W * (TL::STATES / 2);
        const int per = dir ? TL::YA - 1 : TL::XA - 1, line = f / per, a = f - line * per + (W ? 0 : 1);
        const int t0 = (dir ? j0 : i0) - 3 + a + W, k = (dir ? i0 : j0) - 1 + line;
        if (t0 + 2 > (dir ? I.Ny : I.Nx) + 1 || k > (dir ? I.Nx : I.Ny)) continue;   // of no cell of the grid
        SlotAt at;
        at.dir = dir; at.w = W; at.t0 = t0; at.k = k;
        const V3 v = slot_state(I, st, at, -1000, -1000, 0, 0.0);
        double *w = tab + (dir ? TL::XS + (W * TL::YL + line) * TL::YA : (W * TL::XL + line) * TL::XA) + a;
        const int comp = dir ? TL::template comp<1>() : TL::template comp<0>();
        w[0] = v.c[0];
        w[comp] = v.c[dir ? 2 : 1];
        w[2 * comp] = v.c[dir ? 1 : 2];
    }
    __syncthreads();
    const NoHit none;
    for (int e = t; e < FX + FY; e += NT) {
        // the lower face of cell (xi, xj); the last column's or row's upper face is that of the cell after it
        const bool dir = e >= FX;
        const int f = dir ? e - FX : e, xi = dir ? f % kTX : f % (kTX + 1), xj = dir ? f / kTX : f / (kTX + 1);
        const int i = i0 + xi, j = j0 + xj;
        if (i > I.Nx - (dir ? 1 : 0) || j > I.Ny - (dir ? 0 : 1)) continue;
        double z0 = 0.0, z1 = 0.0;
        V3 F;
        H2 hm, hp;
        if (!dir) {
            if constexpr (SURF) {
                const long long x = ((long long)j * (I.Nx + 1) + i) * 2;
                z0 = I.zfx[x];
                z1 = I.zfx[x + 1];
            }
            F = tab_flux<TL, 0, -1, SURF>(tab + xj * TL::XA + xi, none, I.g, hm, hp, z0, z1);
        } else {
            if constexpr (SURF) {
                const long long y = ((long long)j * I.Nx + i) * 2;
                z0 = I.zfy[y];
                z1 = I.zfy[y + 1];
            }
            F = tab_flux<TL, 1, -1, SURF>(tab + xi * TL::YA + xj, none, I.g, hm, hp, z0, z1);
        }
#pragma unroll
        for (int c = 0; c < 3; c++) part[c][e] = F.c[c];
#pragma unroll
        for (int c = 0; c < 2; c++) { part[3 + c][e] = hm.g[c]; part[5 + c][e] = hp.g[c]; }
    }
    __syncthreads();
    if (t >= CELLS) return;                    // the cells' own threads are the first ones
    const int xi = t % kTX, xj = t / kTX, i = i0 + xi, j = j0 + xj;
    double n1 = 0.0;
    if (i < I.Nx && j < I.Ny) {
        double bx[4], by[4], zx[4] = {}, zy[4] = {}, eta = 0.0;
        load_slopes(I, i, j, bx, by);
        if constexpr (SURF) {
            const long long fx = ((long long)j * (I.Nx + 1) + i) * 2, fy = ((long long)j * I.Nx + i) * 2;
#pragma unroll
            for (int q = 0; q < 2; q++) {
                zx[q] = I.zfx[fx + q];
                zx[2 + q] = I.zfx[fx + 2 + q];
                zy[q] = I.zfy[fy + q];
                zy[2 + q] = I.zfy[fy + 2 * I.Nx + q];
            }
            eta = st(0, i, j) + zs[(xj + 2) * kSX + xi + 2];
        }
        const double *const tx = tab + xj * TL::XA + xi, *const ty = tab + xi * TL::YA + xj;
        const int ex = xj * (kTX + 1) + xi, ey = FX + xj * kTX + xi;
        RowParts r;
        auto flux = [&](int e) { return V3{{part[0][e], part[1][e], part[2][e]}}; };
        auto depth = [&](int e, int c) { return H2{{part[c][e], part[c + 1][e]}}; };
        r.fxm = flux(ex); r.fxp = flux(ex + 1); r.fym = flux(ey); r.fyp = flux(ey + kTX);
        r.hx[0] = tab_depth<TL, 0, 1, -2>(tx, none);
        r.hx[1] = depth(ex, 5);
        r.hx[2] = depth(ex + 1, 3);
        r.hx[3] = tab_depth<TL, 0, 0, 1>(tx, none);
        r.hy[0] = tab_depth<TL, 1, 1, -2>(ty, none);
        r.hy[1] = depth(ey, 5);
        r.hy[2] = depth(ey + kTX, 3);
        r.hy[3] = tab_depth<TL, 1, 0, 1>(ty, none);
        const V3 R = row_residual<SURF>(r, I, Recip(I.dx), Recip(I.dy), Recip(I.dx * I.dy), bx, by, zx, zy, eta);
        const long long n = (long long)I.Nx * I.Ny, cidx = (long long)j * I.Nx + i;
        I.R[cidx] = R.c[0];
        I.R[n + cidx] = R.c[1];
        I.R[2 * n + cidx] = R.c[2];
        n1 = fabs(R.c[0]) + fabs(R.c[1]) + fabs(R.c[2]);
        I.rn[cidx] = n1;
    }
    for (int off = 32; off > 0; off >>= 1) n1 += __shfl_down(n1, off, 64);
    if ((t & 63) == 0) red[t >> 6] = n1;
    __syncthreads();
    if (t == 0 && partial) {
        double sum = 0.0;
#pragma unroll
        for (int w = 0; w < NW; w++) sum += red[w];
        partial[blockIdx.y * gridDim.x + blockIdx.x] = sum;
    }
}

// ---- launchers ---------------------------------------------------------------------------

// fewer cells than fill every compute unit (256) with a 32 x 8 tile: what one workgroup waits for is
// spread over more threads or workgroups instead
static bool few_cells(const Inst2D &I) { return (long long)I.Nx * I.Ny < 256LL * kTX * kTY; }

hipError_t launch_residual2d(const Inst2D &I, double *partial, hipStream_t s)
{
    dim3 grid((I.Nx + kTX - 1) / kTX, (I.Ny + kTY - 1) / kTY);
    const bool surf = I.recon == NMG_RECON_SURFACE;
    auto launch = [&](auto kernel, int nt) { hipLaunchKernelGGL(kernel, grid, dim3(nt), 0, s, I, partial); };
    if (few_cells(I)) surf ? launch(k_residual2d<true, 1024>, 1024) : launch(k_residual2d<false, 1024>, 1024);
    else surf ? launch(k_residual2d<true, 512>, 512) : launch(k_residual2d<false, 512>, 512);
    return hipGetLastError();
}

int residual2d_tiles(int Nx, int Ny) { return ((Nx + kTX - 1) / kTX) * ((Ny + kTY - 1) / kTY); }

template <typename T, int NB, bool SURF>
static hipError_t jacobian2d_t(const Inst2D &I, const Perm2D &P, T *J, T *rhs, T *Dinv, hipStream_t s)
{
    const long long nb = border_rows2d(I.Nx, I.Ny);
    const unsigned groups = (unsigned)((nb + BorderLds<NB>::RPW - 1) / BorderLds<NB>::RPW);
    const int gx = (I.Nx + 7) / 8, tiles = gx * ((I.Ny + 7) / 8);
    // interior and border rows in one launch while their workgroups are at most two rounds of two a
    // compute unit: beyond that the border rows' own launch, of smaller workgroups, is the faster one
    // (256 x 128, J21, 1264 workgroups: 223 us in one launch, 210 in two; J9, 888: 155 and 161)
    if (few_cells(I) && tiles + (long long)groups <= 1024) {
        hipLaunchKernelGGL((k_jacobian2d_small<T, NB, SURF>), dim3(tiles + groups), dim3(kJacNT), 0, s, I, P, J, rhs, Dinv,
                           gx, tiles, nb);
        return hipGetLastError();
    }
    if (few_cells(I))
        hipLaunchKernelGGL((k_jacobian2d<T, NB, SURF, 8, 8>), dim3(gx, (I.Ny + 7) / 8), dim3(kJacNT), 0, s, I, P, J, rhs, Dinv);
    else
        hipLaunchKernelGGL((k_jacobian2d<T, NB, SURF, 32, 8>), dim3((I.Nx + 31) / 32, (I.Ny + 7) / 8), dim3(kJacNT), 0, s,
                           I, P, J, rhs, Dinv);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((k_jacobian2d_border<T, NB, SURF>), dim3(groups), dim3(kBorderThreads), 0, s, I, P, J, rhs, Dinv, nb);
    return hipGetLastError();
}

template <typename T, bool SURF>
static hipError_t jacobian2d_nb(const Inst2D &I, const Perm2D &P, void *J, void *rhs, void *Dinv, int nb, hipStream_t s)
{
    if (nb == 21) return jacobian2d_t<T, 21, SURF>(I, P, (T *)J, (T *)rhs, (T *)Dinv, s);
    return jacobian2d_t<T, 9, SURF>(I, P, (T *)J, (T *)rhs, (T *)Dinv, s);
}

hipError_t launch_jacobian2d(const Inst2D &I, const Perm2D &P, void *J, void *rhs, void *Dinv, int prec,
                             hipStream_t s, int nb)
{
    if (nb != 9 && nb != 21) return hipErrorInvalidValue;
    const bool surf = I.recon == NMG_RECON_SURFACE;
    if (prec == NMG_FP32_MG)
        return surf ? jacobian2d_nb<float, true>(I, P, J, rhs, Dinv, nb, s) : jacobian2d_nb<float, false>(I, P, J, rhs, Dinv, nb, s);
    return surf ? jacobian2d_nb<double, true>(I, P, J, rhs, Dinv, nb, s) : jacobian2d_nb<double, false>(I, P, J, rhs, Dinv, nb, s);
}

}  // namespace nmg
