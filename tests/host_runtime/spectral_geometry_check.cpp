// spectral_geometry over problem sizes and shift tables: every energy is an output
// of exactly one block, the transforms' rows and the sandwich's points fit their LDS,
// and the workspace regions of a pass follow each other within the plan's bytes.
#include <algorithm>
#include <cstdio>
#include <vector>

#include "sse_spectral.h"

using namespace sse;

static int fails = 0, on = 0, pi = 0, total = 0;
#define NEED(c) do { if (!(c)) { printf("line %d: NA=%d NB=%d Norb=%d Nkz=%d NE=%d Nw=%d: %s\n", __LINE__, d.NA, d.NB, d.Norb, d.Nkz, d.NE, d.Nw, #c); ++fails; } } while (0)

int main()
{
    for (int prec : {0, 1, 2, 3})
    for (int ncomp : {1, 2})
    for (int NA : {1, 7, 64, 1024, 20000})
    for (int NB : {1, 4, 50})
    for (int Norb : {1, 3, 10, 13, 16, 17, 30})
    for (int Nkz : {1, 3, 7, 21, 64, 70})
    for (int NE : {1, 9, 64, 399, 1000})
    for (int Nw : {1, 8, 40, 128})
    for (int step : {1, -2, 7}) {
        sse_desc d{};
        d.NA = NA; d.NB = NB; d.Norb = Norb; d.N3D = 3; d.Nkz = Nkz; d.Nqz = (Nkz + 1) / 2;
        d.NE = NE; d.Nw = Nw; d.ncomp = ncomp; d.prec = prec;
        std::vector<int32_t> s(Nw);
        for (int w = 0; w < Nw; ++w)
            s[w] = NE > 1 ? step * w % (NE - 1) : 0;
        SpectralGeom g = spectral_geometry(d, s.data());
        ++total;
        NEED(g.on || g.bytes == 0);
        if (!g.on)
            continue;
        ++on;
        const size_t NN = (size_t)Norb * Norb, row = (size_t)g.npt * 16;
        NEED(Norb <= speck::kMaxNorb && g.L == g.r1 * g.r2 && g.L <= 288 && g.npt == Nkz * g.L);
        NEED(g.V == g.L - (g.smax - g.smin) && g.V >= 1);
        NEED(g.V * g.nblk >= NE && g.V * (g.nblk - 1) < NE);
        for (int w = 0; w < Nw; ++w)
            NEED(g.smax - s[w] >= 0 && g.smax - s[w] + g.V <= g.L);
        NEED(g.C == 1 << g.logC && g.rowp >= (g.r1 - 1) * (g.r2 + 1) + g.r2);
        NEED(((size_t)g.L + Nkz + (size_t)Nkz * g.C * g.rowp) * 16 == g.fft_lds && g.fft_lds <= speck::kLdsOne);
        NEED(g.fft_threads % 64 == 0 && g.fft_threads >= 64 && g.fft_threads <= speck::kFftBlock);
        NEED(g.P * g.npg >= g.npt && g.P * (g.npg - 1) < g.npt && g.matrix == speck::matrix_form(Norb));
        if (g.matrix) {
            const int cap = std::min(d.NB, speck::matrix_neighbours(Norb));
            NEED(cap >= 1 && g.P % 16 == 0 && (g.P == 16 || cap == d.NB));  // rounds only with every neighbour staged
            NEED(g.sand_lds == cap * speck::matrix_bytes(Norb, g.P) && g.sand_lds <= speck::kLdsTwo);
        } else {
            NEED(g.P == speck::kSandBlock / Norb);
            NEED(g.sand_lds == NN * g.P * 16 + 3 * NN * 8 && g.sand_lds <= speck::kLdsOne);
        }
        NEED(g.nc >= 1 && g.nc <= ncomp && g.nb >= 1 && g.nb <= g.nblk && g.na >= 1 && g.na <= NA);
        NEED(g.off_dht >= 256 && ((size_t)Nw * 9 + g.L + d.Nqz) * 16 <= speck::kLdsOne);
        NEED(g.off_d >= g.off_dht + NA * NB * 3 * NN * 8);
        NEED(g.off_g >= g.off_d + g.nc * ((size_t)NA * NB * 9 * row));
        NEED(g.off_s >= g.off_g + (size_t)g.nc * g.nb * NA * NN * row);
        NEED(g.bytes >= g.off_s + (size_t)g.nc * g.nb * g.na * NN * row);
        NEED(g.bytes <= speck::kHardBytes && ((g.off_dht | g.off_d | g.off_g | g.off_s) & 15) == 0);
        if (SpectralGeom h = spectral_pi_geometry(d, s.data()); h.on) {
            ++pi;
            const size_t hrow = (size_t)h.npt * 16;
            NEED(prec == 0 && h.V * h.nblk >= NE && h.npt == Nkz * h.L && h.na == NA);
            NEED(h.P * h.npg >= h.npt && h.P * (h.npg - 1) < h.npt && h.matrix == speck::matrix_form(Norb));
            if (h.matrix)
                NEED(h.P % 16 == 0 && h.sand_lds <= speck::kLdsTwo &&
                     h.sand_lds == speck::matrix_tiles(Norb) * 128 * (size_t)std::min(d.NB, speck::pi_matrix_neighbours(Norb)));
            else
                NEED(h.sand_lds >= (size_t)std::max(Norb, 9) * Norb * h.P * 16 + 3 * NN * 8 && h.sand_lds <= speck::kLdsOne);
            NEED(((size_t)h.L + (size_t)Nkz * (h.L + 2 + Nw)) * 16 <= speck::kLdsOne);
            NEED(h.off_g >= h.off_d + h.nc * ((size_t)NA * NB * 9 * hrow));
            NEED(h.off_s >= h.off_g + (size_t)h.nc * h.nb * NA * NN * hrow);
            NEED(h.bytes >= h.off_s + (size_t)h.nc * h.nb * NA * NN * hrow && h.bytes <= speck::kHardBytes);
        }
        d.tile_e = 2;
        NEED(!spectral_geometry(d, s.data()).on);
    }
    printf("%d of %d problems take the spectral form, %d failures\n", on, total, fails);
    if (!fails && on > 1000 && pi > 1000)
        printf("OK\n");
    return fails != 0;
}
