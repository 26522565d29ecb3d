// The pinned slots through which sampling calls read their results, with the HIP
// runtime's calls replaced by the ones below (no GPU): calls on a stream that is
// being captured fail, as the runtime's synchronisation does there, and must not
// use up the slots of the calls after them.
#include <stdio.h>
#include <stdlib.h>
#include <string.h>

#include "../../include/lbm.h"

static int g_capturing, g_copies, g_pinned;

extern "C" {
int hipGetDevice(int *d) { *d = 0; return 0; }
int hipGetLastError(void) { return 0; }
int hipHostMalloc(void **p, size_t n, unsigned) { ++g_pinned; *p = calloc(1, n); return 0; }
int hipStreamIsCapturing(void *, int *s) { *s = g_capturing; return 0; }
int hipThreadExchangeStreamCaptureMode(int *) { return 0; }
int hipStreamSynchronize(void *) { return g_capturing ? 900 : 0; }
int hipMemcpyAsync(void *to, const void *, size_t n, int, void *) { ++g_copies; memset(to, 0, n); return 0; }
// no kernel is launched, on a machine with a GPU either
struct Dim3 { unsigned x, y, z; };
int __hipPushCallConfiguration(Dim3, Dim3, size_t, void *) { return 1; }
int hipLaunchKernel(const void *, Dim3, Dim3, void **, size_t, void *) { return 1; }
}

int main()
{
    lbm_params p;
    memset(&p, 0, sizeof p);
    p.nx = p.ny = 64;
    p.model = LBM_CIL;
    p.tau = 1.0;
    p.A = 0.125;
    p.B = 0.3;
    lbm_ctx *c = nullptr;
    if (lbm_create(&p, (void *)256, (void *)512, 64, nullptr, (void *)4096, 1u << 30, nullptr, &c) != LBM_OK) {
        printf("lbm_create: %s\n", lbm_last_error());
        return 1;
    }
    int bad = 0;
    lbm_obs o;
    auto expect = [&](bool ok, const char *what) {
        if (!ok) {
            printf("unexpected: %s (%s)\n", what, lbm_last_error());
            bad = 1;
        }
    };
    expect(lbm_moments(c, nullptr, nullptr, nullptr, &o) == LBM_OK && g_copies == 0 && g_pinned == 1, "a call's slot");
    g_capturing = 1;
    for (int k = 0; k < 1100; ++k)
        expect(lbm_moments(c, nullptr, nullptr, nullptr, &o) == LBM_EHIP, "a call under capture");
    g_capturing = 0;
    g_copies = 0;
    expect(lbm_moments(c, nullptr, nullptr, nullptr, &o) == LBM_OK && g_copies == 0, "the slots after captures");
    // every slot at once: none was left behind
    lbm_obs *out = (lbm_obs *)calloc(1024, sizeof(lbm_obs));
    const size_t need = lbm_sweep_workspace_bytes(&p, 1, 1024);
    expect(need > 0 && lbm_sweep_samples(&p, 1, 1024, (void *)4096, nullptr, out) == LBM_OK && g_copies == 0,
           "all the slots");
    expect(lbm_sweep_samples(&p, 1, 1, (void *)4096, nullptr, out) == LBM_OK && g_copies == 0, "given back");
    free(out);
    expect(g_pinned == 1, "one page");
    lbm_destroy(c);
    printf(bad ? "host slots: FAILED\n" : "host slots: ok\n");
    return bad;
}
