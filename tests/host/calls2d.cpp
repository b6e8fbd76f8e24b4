// The 2D entry points' host code with the launches recorded instead of made: one query a line on
// standard input,
//   entry nx ny levels jac precision nu1 nu2 nu3 cut capturing cus
// (entry: vcycle, setup or step; cut: bytes the workspace is short of nmg_workspace_bytes; capturing:
// the stream is being captured; cus: compute units of the device), one line a launch on standard
// output and a last one with the call's status.  The planning functions are the library's own.
// The entry `order` (nx and ny as above, then the tile's two sizes) checks instead that a level's rows in
// tiles have a slot each, colour by colour and tile by tile without gaps.
#include <cstdio>
#include <iostream>
#include <string>

#include "api2d.hip"

static int g_cus = 256;
static bool g_capturing = false;

extern "C" {
hipError_t hipStreamIsCapturing(hipStream_t, hipStreamCaptureStatus *st)
{
    *st = g_capturing ? hipStreamCaptureStatusActive : hipStreamCaptureStatusNone;
    return hipSuccess;
}
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipMemcpyAsync(void *, const void *, size_t, hipMemcpyKind, hipStream_t) { return hipSuccess; }
hipError_t hipEventCreate(hipEvent_t *) { return hipSuccess; }
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float *, hipEvent_t, hipEvent_t) { return hipSuccess; }
const char *hipGetErrorString(hipError_t) { return ""; }
}

namespace nmg {

nmg_status set_error(nmg_status st, const char *msg)
{
    fprintf(stderr, "%s\n", msg);
    return st;
}

static hipError_t coop(const char *kind, const Level2D &L, const Resident2D &G, int nu, int prolong, int restr, unsigned tag)
{
    printf("%s %d %d %d %d %d %d %d %d %d %d %d %d %d %u %d\n", kind, L.nx, L.ny, L.nb, L.P.C, G.tx, G.ty, G.gx, G.gy, G.m, nu,
           prolong, restr, (int)(L.P.tw() > 0), tag, (int)resident2d_exchanges(L, nu, G.m));
    return hipSuccess;
}
int resident2d_max_wg(int, int) { return g_cus; }
int streamed2d_max_wg(int) { return g_cus; }
hipError_t launch_resident2d(void *, const Level2D &L, const Level2D &, const Resident2D &G, int nu, int prolong, int restr,
                             unsigned tag, double, void *, long long, const NewtonState *, int, hipStream_t)
{
    return coop("resident", L, G, nu, prolong, restr, tag);
}
hipError_t launch_streamed2d(void *, const Level2D &L, const Level2D &, const Resident2D &G, int nu, int prolong, int restr,
                             unsigned tag, double, void *, long long, const NewtonState *, int, hipStream_t)
{
    return coop("streamed", L, G, nu, prolong, restr, tag);
}
static hipError_t plain(const char *kind, const Level2D &L)
{
    printf("%s %d %d %d\n", kind, L.nx, L.ny, (int)(L.P.tw() > 0));
    return hipSuccess;
}
hipError_t launch_smooth2d_pass(void *, const Level2D &L, int, int, double, int, hipStream_t, int) { return plain("pass", L); }
hipError_t launch_restrict2d(void *, const Level2D &L, const Level2D &, int, hipStream_t) { return plain("restrict", L); }
hipError_t launch_prolong2d(void *, const Level2D &L, const Level2D &, int, hipStream_t) { return plain("prolong", L); }
hipError_t launch_permute2d(const void *, int, void *, int, const Level2D &L, int, int rows, int, hipStream_t)
{
    return plain(rows ? "rows" : "permute", L);
}
hipError_t launch_dinv2d(const double *, void *, const Level2D &, int, hipStream_t) { return hipSuccess; }
hipError_t launch_coarsen2d(void *, const Level2D &, const Level2D &, int, hipStream_t) { return hipSuccess; }
hipError_t launch_coarse_factor2d(void *, const Level2D &, double *, int, hipStream_t) { return hipSuccess; }
hipError_t launch_bottom2d(void *, const Level2D *, int, int, int, int, double, const double *, int, hipStream_t, int) { return hipSuccess; }
hipError_t launch_sweeps2d(void *, const Level2D &, int, double, int, hipStream_t) { return hipSuccess; }
hipError_t launch_fill(void *, int, long long, hipStream_t) { return hipSuccess; }
hipError_t launch_update2d(double *, const void *, const Level2D &, double, const NewtonState *, int, hipStream_t) { return hipSuccess; }
hipError_t launch_residual2d(const Inst2D &, double *, hipStream_t) { return hipSuccess; }
hipError_t launch_jacobian2d(const Inst2D &, const Perm2D &, void *, void *, void *, int, hipStream_t, int) { return hipSuccess; }
hipError_t launch_state2d(const double *, int, long long, double, int, NewtonState *, double *, int, int, hipStream_t) { return hipSuccess; }
hipError_t launch_sum_res(const double *, int, double *, hipStream_t) { return hipSuccess; }

}  // namespace nmg

// 0 if the rows of every tile and colour are numbered one after the other from tile3_start, and the
// next tile's begin where they end
static int bad_order(int nx, int ny, int tw, int th)
{
    using namespace nmg;
    Perm2D P = make_perm2d(nx, ny, 3);
    tile_rows(P, nx, tw, th);
    for (int c = 0; c < 3; c++) {
        long long next = (long long)c * P.ny * P.W;
        for (int j0 = 0; j0 < ny; j0 += th)
            for (int i0 = 0; i0 < nx; i0 += tw) {
                const int w = std::min(tw, nx - i0), h = std::min(th, ny - j0);
                if (tile3_start(P, c, i0, j0, h) != next) return 1;
                int e = 0;
                for (int jr = 0; jr < h; jr++)
                    for (int il = 0; il < w; il++) {
                        if ((i0 + il + j0 + jr) % 3 != c) continue;
                        int i = -1, j = -1;
                        tile3_cell(c, i0, j0, w, e, i, j);
                        if (i != il || j != jr || perm2d_rows(P, i0 + il, j0 + jr) != next + e) return 2;
                        e++;
                    }
                if (e != tile3_count(c, i0, j0, w, h)) return 3;
                next += e;
            }
        if (next > (long long)(c + 1) * P.ny * P.W) return 4;
    }
    return 0;
}

int main()
{
    std::string entry;
    nmg_desc d;
    nmg_params p;
    long long cut;
    int capturing;
    memset(&d, 0, sizeof(d));
    memset(&p, 0, sizeof(p));
    d.dim = 2;
    d.x1 = d.y1 = 1.0;
    d.g = 9.8;
    d.bx_gp = d.by_gp = (const double *)8;       // placeholders, never read
    for (int k = 0; k < 4; k++) d.bc[k].kind = NMG_BC_EXTRAP;
    p.eps = 1e-6;
    p.tau = p.omega = 1.0;
    p.n_max = 10;
    p.check_every = 1;
    void *const any = (void *)256;               // as are the buffers and the stream
    while (std::cin >> entry >> d.nx >> d.ny) {
        if (entry == "order") {
            int tw, th;
            std::cin >> tw >> th;
            printf("end %d\n", bad_order(d.nx, d.ny, tw, th));
            continue;
        }
        std::cin >> d.levels >> d.jac >> p.precision >> p.nu1 >> p.nu2 >> p.nu3 >> cut >> capturing >> g_cus;
        g_capturing = capturing != 0;
        const size_t bytes = nmg::workspace2d_bytes(&d, &p) - (size_t)cut;
        nmg_status st;
        if (entry == "step") st = nmg::newton2d_steps(&d, &p, any, bytes, (double *)any, 1, nullptr, (hipStream_t)64);
        else st = nmg::vcycle2d(&d, &p, any, bytes, any, any, any, entry == "setup", (hipStream_t)64);
        printf("end %d\n", (int)st);
    }
    return 0;
}
