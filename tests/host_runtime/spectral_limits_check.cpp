// Launch sizes of the spectral form where an instance has many atoms or neighbours and
// little else: fewer than 2^32 threads in every launch; and the geometry that a device test
// stands on.
#include <algorithm>
#include <cstdio>
#include <vector>

#include "sse_spectral.h"

using namespace sse;

static int fails = 0, on = 0, pi = 0;
#define NEED(c) do { if (!(c)) { printf("line %d: NA=%d NB=%d Norb=%d Nkz=%d NE=%d Nw=%d: %s\n", __LINE__, d.NA, d.NB, d.Norb, d.Nkz, d.NE, d.Nw, #c); ++fails; } } while (0)

static const int64_t kMost = 0xffffffffLL;

int main()
{
    for (int NA : {20000, 50000, 80000, 200000, 1000000, 4000000})
    for (int NB : {1, 4, 50})
    for (int Norb : {1, 2, 4, 7, 10})
    for (int Nkz : {1, 3, 7})
    for (int NE : {6, 10, 60})
    for (int Nw : {1, 4}) {
        sse_desc d{};
        d.NA = NA; d.NB = NB; d.Norb = Norb; d.N3D = 3; d.Nkz = d.Nqz = Nkz;
        d.NE = NE; d.Nw = Nw; d.ncomp = 2;
        std::vector<int32_t> s(Nw);
        for (int w = 0; w < Nw; ++w)
            s[w] = w + 1;
        const int64_t ab = (int64_t)NA * NB, NN = (int64_t)Norb * Norb;
        auto transform = [&](const SpectralGeom &g, int threads) {
            return (NA * NN + g.C - 1) / g.C * g.nb * threads;
        };
        auto sandwich = [&](const SpectralGeom &g, int nb) {
            return (int64_t)(NA + 7) / 8 * 8 * g.npg * nb * speck::kSandBlock;
        };
        if (SpectralGeom g = spectral_geometry(d, s.data()); g.on) {
            ++on;
            const int64_t dhat = ab * Nkz * speck::kSandBlock;
            NEED(dhat + 512 * speck::kSandBlock <= kMost);
            NEED(transform(g, std::max(g.fft_threads, speck::kSandBlock)) <= kMost);
            NEED(sandwich(g, g.nb) <= kMost);
        }
        if (SpectralGeom g = spectral_pi_geometry(d, s.data()); g.on) {
            ++pi;
            NEED(2 * transform(g, g.fft_threads) + 512 * g.fft_threads <= kMost);
            NEED(sandwich(g, 1) <= kMost);
            NEED(ab * 9 * speck::kSandBlock <= kMost);
        }
    }
    {
        // the device test of a workspace of some atoms at a time has three passes, the last one ragged
        sse_desc d{};
        d.NA = 900; d.NB = 4; d.Norb = 16; d.N3D = 3; d.Nkz = d.Nqz = 9; d.NE = 140; d.Nw = 20; d.ncomp = 1;
        std::vector<int32_t> s(d.Nw);
        for (int w = 0; w < d.Nw; ++w)
            s[w] = w + 1;
        const SpectralGeom g = spectral_geometry(d, s.data());
        NEED(g.on && !g.matrix && g.na == 425 && g.nb == 1);
    }
    printf("%d and %d problems in the spectral form, %d failures\n", on, pi, fails);
    if (!fails && on > 100 && pi > 100)
        printf("OK\n");
    return fails != 0;
}
