// A plan begun on a stream that is being captured, with the built library over a stand-in for the HIP
// runtime: device memory is host memory, a copy on a captured stream is recorded and not made, a
// wait for such a stream is refused, launches do nothing.  Prints, one a line: the status of a begin
// under capture, the bytes of the copies recorded meanwhile, the status and the copied bytes of the
// first begin after it, and the same two of a plan that was never captured.
#include <hip/hip_runtime.h>

#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <vector>

#include "nmg.h"

static bool g_capturing = false;
static size_t g_recorded = 0, g_copied = 0;

extern "C" {
hipError_t hipStreamIsCapturing(hipStream_t, hipStreamCaptureStatus *st)
{
    *st = g_capturing ? hipStreamCaptureStatusActive : hipStreamCaptureStatusNone;
    return hipSuccess;
}
hipError_t hipStreamSynchronize(hipStream_t) { return g_capturing ? hipErrorStreamCaptureUnsupported : hipSuccess; }
hipError_t hipMemcpyAsync(void *to, const void *from, size_t n, hipMemcpyKind, hipStream_t)
{
    (g_capturing ? g_recorded : g_copied) += n;
    if (!g_capturing) memcpy(to, from, n);
    return hipSuccess;
}
hipError_t hipHostMalloc(void **p, size_t n, unsigned) { return (*p = malloc(n)) ? hipSuccess : hipErrorOutOfMemory; }
hipError_t hipLaunchKernel(const void *, dim3, dim3, void **, size_t, hipStream_t) { return hipSuccess; }
hipError_t hipGetLastError(void) { return hipSuccess; }
const char *hipGetErrorString(hipError_t) { return "refused"; }
}

int main()
{
    nmg_desc d;
    nmg_params p;
    memset(&d, 0, sizeof(d));
    memset(&p, 0, sizeof(p));
    d.dim = 1;
    d.nx = 12800;
    d.ny = 1;
    d.levels = 8;
    d.jac = 3;
    d.x1 = 1.0;
    d.g = 9.8;
    d.sig_face = d.sig_gp = d.sigx_gp = d.bx_gp = (const double *)8;   // placeholders, never read
    p.eps = 1e-2;
    p.tau = p.omega = 1.0;
    p.nu1 = p.nu2 = p.nu3 = 2;
    p.n_max = 10;
    p.check_every = 1;
    std::vector<double> U(2 * d.nx, 1.0);
    double *states[1] = {U.data()};
    auto begin = [&](nmg_plan *plan, std::vector<char> &ws) {
        return (int)nmg_plan_begin(plan, ws.data(), ws.size(), states, (void *)64);   // any stream but the null one
    };
    nmg_plan *a = nullptr, *b = nullptr;
    if (nmg_plan_create(&d, &p, 1, &a) != NMG_OK || nmg_plan_create(&d, &p, 1, &b) != NMG_OK) return 1;
    std::vector<char> wa(nmg_plan_workspace_bytes(a)), wb(nmg_plan_workspace_bytes(b));
    g_capturing = true;
    printf("%d\n", begin(a, wa));
    printf("%zu\n", g_recorded);
    g_capturing = false;
    printf("%d\n", begin(a, wa));
    printf("%zu\n", g_copied);
    g_copied = 0;
    printf("%d\n", begin(b, wb));
    printf("%zu\n", g_copied);
    nmg_plan_destroy(a);
    nmg_plan_destroy(b);
    return 0;
}
