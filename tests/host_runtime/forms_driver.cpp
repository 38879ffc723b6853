// Which form a submission runs and what workspace its kernels get: the runtime with
// stand-in launchers of the spectral form.  argv[1] names the check; exits non-zero on
// failure.
#include <cstdint>
#include <cstdio>
#include <cstring>
#include <vector>

#include "sse_spectral.h"

using namespace sse;

static int n_spectral = 0;

// What the kernels of one instance may touch lies in the caller's workspace.
static char *g_ws = nullptr;
static size_t g_ws_bytes = 0;
static bool g_bad = false;
static void touch(const SpectralGeom &g, const sse_desc &d, char *ws)
{
    const size_t row = (size_t)g.npt * 16 * d.Norb * d.Norb;
    const size_t end = g.off_s + (size_t)g.nc * g.nb * g.na * row;
    // complex values lie on their own size, 16 bytes
    if (((uintptr_t)ws | g.off_dht | g.off_d | g.off_g | g.off_s) & 15)
        g_bad = true;
    if (ws < g_ws + 4 || ws + end > g_ws + g_ws_bytes)
        g_bad = true;
}

namespace sse {
hipError_t spectral_sigma_launch(const sse_desc &d, const SpectralGeom &g, const int32_t *, const sse_args &,
                                 uint32_t *status, bool clear, uint32_t *host, const Fp64Params &, size_t, void *ws,
                                 hipStream_t)
{
    ++n_spectral;
    touch(g, d, (char *)ws);
    if (clear)
        *status = 0;
    if (host)
        *host = *status;
    return hipSuccess;
}
hipError_t spectral_batch_launch(int n, const sse_desc *const *d, const SpectralGeom *const *g, const sse_args *const *,
                                 const size_t *off, const SpecParams *, const SpecParams *, const Fp64Params *, size_t,
                                 uint32_t *status, bool clear, char *ws, hipStream_t)
{
    ++n_spectral;
    for (int i = 0; i < n; ++i)
        touch(*g[i], *d[i], ws + off[i]);
    if (clear)
        *status = 0;
    return hipSuccess;
}
hipError_t spectral_pi_launch(const sse_desc &d, const SpectralGeom &g, const int32_t *, const int32_t *,
                              const double *, const void *, void *, uint32_t *, void *ws, hipStream_t)
{
    ++n_spectral;
    touch(g, d, (char *)ws);
    return hipSuccess;
}
}  // namespace sse

static sse_desc desc(int prec, int chunk_taps)
{
    sse_desc d{};
    d.NA = 16; d.NB = 4; d.Norb = 10; d.N3D = 3; d.Nkz = 3; d.Nqz = 3; d.NE = 41; d.Nw = 6;
    d.ncomp = 2; d.prec = prec; d.alpha_im = 1; d.chunk_taps = chunk_taps;
    return d;
}
static const int32_t kShift[6] = {1, 2, 3, 4, 5, 6};
static int32_t kNeigh[64];
static double one[1];

// The form that a batch of two runs in a workspace of `bytes`: 1 spectral, 0 direct, -1 refused.
static int batch_form(sse_plan_t p, size_t bytes)
{
    std::vector<char> w(bytes);
    g_ws = w.data();
    g_ws_bytes = bytes;
    n_spectral = 0;
    sse_args a[2] = {{kNeigh, one, one, one, one}, {kNeigh, one, one, one, one}};
    uint64_t t;
    if (sse_submit(p, a, w.data(), bytes, nullptr, &t))
        return -1;
    return sse_wait(t) ? -2 : n_spectral > 0;
}

static int batch_in_a_direct_workspace()
{
    for (int prec : {SSE_FP64, SSE_FP64C64}) {
        const int32_t *sh[2] = {kShift, kShift};
        sse_desc free2[2] = {desc(prec, 0), desc(prec, 0)}, direct2[2] = {desc(prec, 128), desc(prec, 128)};
        sse_plan_t p, pd;
        size_t full, least;
        if (sse_plan_batch(free2, sh, 2, &p, &full) || sse_plan_batch(direct2, sh, 2, &pd, &least))
            return 1;
        if (least >= full || batch_form(p, full) != 1 || batch_form(pd, least) != 0)
            return 2;
        if (batch_form(p, least) != 0 || batch_form(p, full - 1) != 0)
            return 3;
        if (batch_form(p, least - 1) != -1)
            return 4;
        sse_plan_destroy(p);
        sse_plan_destroy(pd);
    }
    return 0;
}

// Workspaces that start 4, 8 and 252 bytes behind a multiple of 256 (the status word alone
// wants four): single plans, a batch and Pi, in the plan's own size.
static int workspace_at_any_word()
{
    for (int off : {0, 4, 8, 252}) {
        const int32_t *sh[2] = {kShift, kShift};
        sse_desc d = desc(SSE_FP64, 0), d2[2] = {d, d};
        sse_plan_t p, pb;
        size_t n, nb;
        if (sse_plan(&d, kShift, &p, &n) || sse_plan_batch(d2, sh, 2, &pb, &nb))
            return 1;
        const size_t most = n > nb ? n : nb;
        std::vector<char> w(most + 512);
        char *base = (char *)(((uintptr_t)w.data() + 255) & ~(uintptr_t)255) + off;
        sse_args a[2] = {{kNeigh, one, one, one, one}, {kNeigh, one, one, one, one}};
        uint64_t t[3];
        n_spectral = 0;
        g_ws = base;
        g_ws_bytes = n;
        if (sse_submit(p, a, base, n, nullptr, &t[0]) || sse_wait(t[0]))
            return 2;
        if (sse_pi_submit(p, kNeigh, one, one, one, base, n, nullptr, &t[1]))
            return 3;
        sse_wait(t[1]);  // the stand-in of the last kernel delivers no status
        g_ws_bytes = nb;
        if (sse_submit(pb, a, base, nb, nullptr, &t[2]) || sse_wait(t[2]))
            return 4;
        if (n_spectral != 3)
            return 5;
        sse_plan_destroy(p);
        sse_plan_destroy(pb);
    }
    return 0;
}

int main(int argc, char **argv)
{
    int r = -1;
    if (argc > 1 && !strcmp(argv[1], "batch_in_a_direct_workspace"))
        r = batch_in_a_direct_workspace();
    if (argc > 1 && !strcmp(argv[1], "workspace_at_any_word"))
        r = workspace_at_any_word();
    if (r == 0 && !g_bad)
        printf("OK\n");
    else
        printf("%s: %d %s\n", argc > 1 ? argv[1] : "?", r, sse_last_error());
    return r != 0 || g_bad;
}
