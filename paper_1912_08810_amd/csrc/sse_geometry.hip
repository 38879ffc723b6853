// sse_geometry.hip -- host-side tile geometry of the kernels: energies per
// tile, tap chunks whose G window fits the LDS budget, MFMA tap groups, LDS
// bytes and workspace sizes.  Host code only (also built by the host-side
// runtime test with a stand-in HIP header).
#include <algorithm>
#include <cmath>
#include <vector>

#include "sse_internal.h"
#include "sse_mfma.h"
#include "sse_spectral.h"

namespace sse {

TileGeom fp64_geometry(int Norb, int NE, const TapTable &taps, int te_request, int chunk_cap,
                       TapTable *out)
{
    const int NN = Norb * Norb;
    int TE = fp64k::kPmax / NN;
    if (te_request > 0)
        TE = std::min(TE, te_request);
    TE = std::max(1, std::min(TE, NE));
    const size_t a_bytes = (size_t)kN3D * NN * sizeof(double);
    const long budget = (long)((fp64k::kLdsBudget - a_bytes) / sizeof(double2));

    *out = taps;
    out->nchunk = 0;
    int t = 0;
    long win_max = 0;
    while (t < taps.n) {
        int u = t + 1;
        while (u < taps.n && (chunk_cap <= 0 || u - t < chunk_cap) &&
               fp64k::kPmax + (long)(taps.s[t] - taps.s[u]) * NN <= budget)
            ++u;
        out->cb[out->nchunk++] = t;
        win_max = std::max(win_max, fp64k::kPmax + (long)(taps.s[t] - taps.s[u - 1]) * NN);
        t = u;
    }
    out->cb[out->nchunk] = taps.n;
    TileGeom g;
    g.TE = TE;
    g.n_etiles = (NE + TE - 1) / TE;
    g.lds_win = (int)std::max(win_max, (long)kN3D * TE * NN);
    g.lds_bytes = (size_t)g.lds_win * sizeof(double2) + a_bytes;
    return g;
}

void fill_tap_pairs(Fp64Params &p)
{
    for (int t = 0; t < 2 * kMaxTaps + 4; ++t)
        p.tws[t] = 0;
    for (int t = 0; t < p.taps.n; ++t) {
        p.tws[2 * t] = p.taps.w[t];
        p.tws[2 * t + 1] = p.taps.s[t];
    }
}

TileGeom mfma_geometry(int Norb, int NE, const TapTable &taps, int te_request, int chunk_cap,
                       TapTable *out, GroupTable *groups)
{
    const int NN = Norb * Norb;
    int TE = mfmak::kPwg / NN;
    if (te_request > 0)
        TE = std::min(TE, te_request);
    TE = std::max(1, std::min(TE, NE));
    // the sandwich's LDS region and output tiles per wave bound TE too (small
    // Norb only: Norb >= 4 keeps TE = kPwg / Norb^2)
    while (TE > 1 && (mfmak::sand_bytes(Norb, TE) > mfmak::kSandBytes ||
                      mfmak::sand_tiles(Norb, TE) > 8 * mfmak::kSandT))
        --TE;
    // A plane holds the window rows plus the reach of the columns past the
    // tile's last position: kPwg + (shift spread of the chunk) NN words; a
    // chunk's A fragments fill at most kMaxG groups.
    *out = taps;
    out->nchunk = 0;
    groups->n = 0;
    int t = 0;
    long win_max = 0;
    while (t < taps.n) {
        int u = t + 1;
        while (u < taps.n && u - t < mfmak::kMaxG * mfmak::kGS &&
               (chunk_cap <= 0 || u - t < chunk_cap) &&
               mfmak::kPwg + (long)(taps.s[t] - taps.s[u]) * NN <= mfmak::kPlaneWords)
            ++u;
        groups->gb[out->nchunk] = groups->n;
        for (int g = t; g < u; g += mfmak::kGS)
            groups->t0[groups->n++] = g;
        out->cb[out->nchunk++] = t;
        win_max = std::max(win_max, (long)(TE + taps.s[t] - taps.s[u - 1]) * NN);
        t = u;
    }
    out->cb[out->nchunk] = taps.n;
    groups->gb[out->nchunk] = groups->n;
    TileGeom g;
    g.TE = TE;
    g.n_etiles = (NE + TE - 1) / TE;
    g.lds_win = (int)win_max;
    g.lds_bytes = 0;  // static LDS: two window buffers and the sandwich region
    return g;
}

size_t mfma_afrag_bytes(int, int NA, int NB, int Nqz, const GroupTable &g)
{
    return (size_t)NA * NB * Nqz * g.n * 64 * 32;
}

size_t mfma_split_offset(int prec, int NA, int NB, int Nqz, const GroupTable &g)
{
    return (mfmak::kZeroPage + mfma_afrag_bytes(prec, NA, NB, Nqz, g) + 255) & ~(size_t)255;
}

size_t mfma_aux_bytes(int prec, int NA, int NB, int Nqz, int Nkz, int NE, int Norb,
                      const GroupTable &g)
{
    size_t b = mfma_split_offset(prec, NA, NB, Nqz, g);
    if (prec == SSE_BF16X3)
        b += (size_t)Nkz * NE * NA * Norb * Norb * 8;
    return b;
}

// Geometry of the phonon kernel (sse_pi.hip): the most neighbours per
// workgroup (up to 4) whose buffers leave room for a ring of the taps' rows,
// then the taps, sorted by increasing shift, cut into chunks of at most 32
// whose ring fits.  LDS per workgroup: ring R + 2 rows (a step's R rows, a
// spare for the next step's top row, a zero row) of NNp (the pairs padded to an
// even count) complex128 values; Zb NNp rows of 16 ntn binary64 columns;
// per neighbour U (3 blocks) and Y (1 block) complex128 and dH (3 blocks) binary64.
PiGeom pi_geometry(int Norb, int NB, const int32_t *w_shift, int Nw)
{
    PiGeom gm{};
    const size_t NN = (size_t)Norb * Norb, NNp = NN + (NN & 1);
    std::vector<int> order(Nw);
    for (int w = 0; w < Nw; ++w)
        order[w] = w;
    std::stable_sort(order.begin(), order.end(),
                     [&](int x, int y) { return w_shift[x] < w_shift[y]; });
    for (int t = 0; t < Nw; ++t) {
        gm.tw[t] = order[t];
        gm.ts[t] = w_shift[order[t]];
    }
    auto ntn_of = [](int nbw) { return (nbw * 9 * 2 + 15) / 16; };
    auto fixed_of = [&](int nbw) {
        return 2 * NNp * 16 + NNp * 16 * ntn_of(nbw) * 8 + (size_t)nbw * NN * (3 * 16 + 16 + 3 * 8);
    };
    const size_t per_row = NNp * 16;
    const size_t budget = pik::kLdsBudgetOne;
    const int want_rows = std::min(gm.ts[Nw - 1] - gm.ts[0] + 1, 8);
    int rmax = 0;
    for (gm.nbw = std::min(NB, pik::kMaxNbw); gm.nbw >= 1; --gm.nbw) {
        const size_t fixed = fixed_of(gm.nbw);
        rmax = fixed < budget ? (int)((budget - fixed) / per_row) : 0;
        if (rmax >= want_rows || gm.nbw == 1)
            break;
    }
    gm.R = 0;
    gm.nchunk = 0;
    int maxtaps = 0;
    int t = 0;
    while (t < Nw && rmax >= 1) {
        int e = t + 1;
        while (e < Nw && e - t < pik::kMaxChunkTaps && gm.ts[e] - gm.ts[t] + 1 <= rmax)
            ++e;
        gm.cb[gm.nchunk] = t;
        gm.R = std::max(gm.R, gm.ts[e - 1] - gm.ts[t] + 1);
        maxtaps = std::max(maxtaps, e - t);
        ++gm.nchunk;
        t = e;
    }
    gm.cb[gm.nchunk] = Nw;
    gm.mtiles = maxtaps <= 16 ? 1 : 2;
    // the final reduction reuses LDS for half the waves' accumulator tiles
    gm.lds_bytes = std::max((size_t)gm.R * per_row + fixed_of(gm.nbw),
                            (size_t)(pik::kWaves / 2) * 16 * gm.mtiles * 16 * ntn_of(gm.nbw) * 8);
    gm.ok = rmax >= 1 && gm.lds_bytes <= budget;
    return gm;
}

SpecParams spectral_params(const sse_desc &d, const SpectralGeom &g, const int32_t *w_shift)
{
    SpecParams p{};
    p.NA = d.NA;
    p.NB = d.NB;
    p.Norb = d.Norb;
    p.NN = d.Norb * d.Norb;
    p.Nkz = d.Nkz;
    p.Nqz = d.Nqz;
    p.NE = d.NE;
    p.Nw = d.Nw;
    p.ncomp = d.ncomp;
    p.L = g.L;
    p.V = g.V;
    p.C = g.C;
    p.logC = g.logC;
    p.rowp = g.rowp;
    p.npt = g.npt;
    p.P = g.P;
    p.npg = g.npg;
    p.smin = g.smin;
    p.smax = g.smax;
    p.nblk = g.nblk;
    p.na_cap = g.na;
    p.antiherm = d.dt_antiherm;
    p.matrix = g.matrix;
    p.g_elems = (int64_t)d.Nkz * d.NE * d.NA * p.NN;
    p.d_elems = (int64_t)d.Nqz * d.Nw * d.NA * d.NB * kNF;
    p.guard_bits = speck::guard_bits(d.prec, d.Norb);
    p.off_suspect = (int64_t)g.off_suspect;
    p.guard_k = (uint32_t)(std::log2((double)d.Nkz) * (1 << 18));
    p.guard_quads = (int64_t)(g.guard_bytes / 16);
    p.off_dht = (int64_t)g.off_dht;
    p.off_d = (int64_t)g.off_d;
    p.off_g = (int64_t)g.off_g;
    p.off_s = (int64_t)g.off_s;
    p.alpha_re = d.alpha_re;
    p.alpha_im = d.alpha_im;
    for (int w = 0; w < d.Nw; ++w)
        p.shift[w] = w_shift[w];
    return p;
}

namespace {

size_t up(size_t x) { return (x + speck::kAlign - 1) & ~(speck::kAlign - 1); }
// At the end of a layout: room for its start to move to a multiple of kAlign, and more.
constexpr size_t kSlack = 4096;

// Workspace layout for the most components, then energy blocks, then sandwich
// atoms per pass that fit budget; false if an eighth of the atoms does not fit.
bool spectral_layout(const sse_desc &d, size_t budget, SpectralGeom *g)
{
    const size_t NN = (size_t)d.Norb * d.Norb, row = (size_t)g->npt * 16;
    const size_t gb = (size_t)d.NA * NN * row, db = (size_t)d.NA * d.NB * kNF * row;
    const size_t peaks = (size_t)d.ncomp * g->nblk * d.NA * NN * 4;
    g->off_suspect = speck::kAlign + peaks;
    g->guard_bytes = up(peaks + (size_t)d.ncomp * d.NA * d.NE * 4);
    const size_t dht = up((size_t)d.NA * d.NB * kN3D * NN * 8);
    const size_t fixed = g->guard_bytes + dht + 4 * speck::kAlign + kSlack;
    for (g->nc = d.ncomp; g->nc >= 1; --g->nc) {
        const size_t base = fixed + g->nc * db, per = 2 * g->nc * gb;
        if (budget < base + (g->nc > 1 ? per : gb + gb / 8))
            continue;
        g->nb = (int)std::min<size_t>(g->nblk, std::max<size_t>(1, (budget - base) / per));
        g->na = d.NA;
        if (base + per > budget)  // one component, one block, some atoms
            g->na = (int)std::max<size_t>(1, (budget - base - gb) / (NN * row));
        g->off_dht = speck::kAlign + g->guard_bytes;  // behind the non-finite flag
        g->off_d = g->off_dht + dht;
        g->off_g = g->off_d + up(g->nc * db);
        g->off_s = g->off_g + up((size_t)g->nc * g->nb * gb);
        g->bytes = g->off_s + up((size_t)g->nc * g->nb * g->na * NN * row) + kSlack;
        return true;
    }
    return false;
}

// The same for Pi: one or both components, then energy blocks; two transforms of G
// per component (X and the opposite Y), every atom.
bool spectral_pi_layout(const sse_desc &d, size_t budget, SpectralGeom *g)
{
    const size_t NN = (size_t)d.Norb * d.Norb, row = (size_t)g->npt * 16;
    const size_t gb = (size_t)d.NA * NN * row, db = (size_t)d.NA * d.NB * kNF * row;
    const size_t dht = up((size_t)d.NA * d.NB * kN3D * NN * 8);
    g->guard_bytes = up((size_t)d.ncomp * d.NA * d.NB * kNF * 4);  // peaks
    const size_t fixed = g->guard_bytes + dht + 4 * speck::kAlign + kSlack;
    // the output pass has a workgroup per (atom, neighbour, i, j), and a launch fewer than 2^32 threads
    if ((int64_t)d.NA * d.NB * kNF * speck::kSandBlock > 0xffffffffLL)
        return false;
    // it holds a transform row per momentum and its sums per frequency
    if (((size_t)g->L + (size_t)d.Nkz * (g->L + 2 + d.Nw)) * 16 > speck::kLdsOne)
        return false;
    for (g->nc = d.ncomp; g->nc >= 1; --g->nc) {
        const size_t base = fixed + g->nc * db, per = 2 * g->nc * gb;
        if (budget < base + per)
            continue;
        g->nb = (int)std::min<size_t>(g->nblk, (budget - base) / per);
        g->na = d.NA;
        g->off_dht = speck::kAlign + g->guard_bytes;
        g->off_d = g->off_dht + dht;
        g->off_g = g->off_d + up(g->nc * db);
        g->off_s = g->off_g + up((size_t)g->nc * g->nb * gb);
        g->bytes = g->off_s + up((size_t)g->nc * g->nb * gb) + kSlack;
        return true;
    }
    return false;
}

// The cheapest transform length whose pass fits: points computed, weighted by what
// the transforms lose.  Of the whole call at Nkz 7, Norb 10, NB 4, complex128, L 256 and
// 288 against 160: one workgroup per CU (64-byte pieces, 115 kB of LDS) 4 % per point,
// 32-byte pieces (two workgroups, 57 kB) 11 %.  Device scale: L 288 in 4 blocks 73 ms,
// L 160 in 8 (a ninth more points) 76 ms.
template <typename Layout>
SpectralGeom best_geometry(const sse_desc &d, const int32_t *w_shift, bool matrix, Layout layout)
{
#define SSE_LENGTH(R1, R2) {R1, R2},
    static const int kSizes[][2] = {SSE_SPECTRAL_LENGTHS(SSE_LENGTH)};
#undef SSE_LENGTH
    SpectralGeom best;
    if (d.Norb > speck::kMaxNorb || d.Nkz > 64)
        return best;
    const int64_t NN = (int64_t)d.Norb * d.Norb;
    if (d.NA * NN > (1 << 28) || (int64_t)d.NA * d.NB > (1 << 28))
        return best;
    int smin = w_shift[0], smax = w_shift[0];
    for (int w = 0; w < d.Nw; ++w) {
        smin = std::min(smin, w_shift[w]);
        smax = std::max(smax, w_shift[w]);
    }
    const bool c64 = d.prec != SSE_FP64;
    double best_cost = 0.0;
    for (const auto &sz : kSizes) {
        SpectralGeom g;
        g.r1 = sz[0];
        g.r2 = sz[1];
        g.L = g.r1 * g.r2;
        g.smin = smin;
        g.smax = smax;
        g.V = g.L - (smax - smin);
        if (g.V < 1)
            continue;
        g.nblk = (d.NE + g.V - 1) / g.V;
        g.npt = d.Nkz * g.L;
        // the matrix form walks its points in rounds of 16, so that a workgroup's start is
        // paid once; rounds as long as 2048 workgroups remain (one GPU's energy shard:
        // 4.53, 4.11 and 4.03 ms per component with 16, 32 and 64 points)
        g.matrix = matrix;
        g.P = matrix ? 16 : speck::kSandBlock / d.Norb;
        while (matrix && g.P < 64 && 2 * g.P <= g.npt && d.NB * speck::matrix_bytes(d.Norb, 2 * g.P) <= speck::kLdsTwo &&
               (int64_t)d.NA * d.ncomp * g.nblk * (g.npt / (2 * g.P)) >= 2048)
            g.P *= 2;
        g.npg = (g.npt + g.P - 1) / g.P;
        g.sand_lds = matrix ? speck::matrix_bytes(d.Norb, g.P) * std::min(d.NB, speck::matrix_neighbours(d.Norb))
                            : (size_t)NN * g.P * 16 + kN3D * NN * 8;
        for (g.logC = 1; g.logC <= 3; ++g.logC) {
            g.C = 1 << g.logC;
            // the rows of a momentum's C channels start 16 / C sixteen-byte banks apart
            // (an odd multiple of that, so that they take all C places)
            g.rowp = g.r1 * (g.r2 + 1);
            while (g.rowp % (32 / g.C) != 16 / g.C)
                ++g.rowp;
            g.fft_lds = ((size_t)g.L + d.Nkz + (size_t)d.Nkz * g.C * g.rowp) * 16;
            if (g.fft_lds > speck::kLdsOne)
                continue;
            const int items = d.Nkz * g.C * g.r2;
            g.fft_threads = std::min(speck::kFftBlock, (items + 63) / 64 * 64);
            if (!layout(d, speck::kSoftBytes, &g) && !layout(d, speck::kHardBytes, &g))
                continue;
            const int piece = g.C * (c64 ? 8 : 16);
            const double cost = (double)g.nblk * g.L * (1.0 + (piece < 64 ? 0.11 : 0.0) + (piece < 32 ? 0.3 : 0.0) +
                                                        (g.fft_lds > speck::kLdsTwo ? 0.04 : 0.0));
            if (best_cost == 0.0 || cost < best_cost) {
                best_cost = cost;
                best = g;
                best.on = true;
            }
        }
    }
    return best;
}

// Estimated microseconds of the spectral form (both self-energies have the same work).
double spectral_us(const sse_desc &d, const SpectralGeom &g)
{
    const double pts = (double)d.Nkz * g.nblk * g.L * d.NA * d.Norb * d.Norb;
    return 25.0 + d.ncomp * (pts * d.NB * (24.0 * d.Norb + 72.0) / 45e6 + pts * 64.0 / 3.5e6);
}

double direct_flops(const sse_desc &d)
{
    return (double)d.Nkz * d.NE * d.NA * d.Norb * d.Norb * d.NB *
           ((d.dt_antiherm ? 36.0 : 72.0) * d.Nqz * d.Nw + 48.0 * d.Norb);
}

}  // namespace

SpectralGeom spectral_geometry(const sse_desc &d, const int32_t *w_shift)
{
    // an explicit tile shape asks for the direct kernel that has tiles
    if (d.tile_e > 0 || d.chunk_taps > 0)
        return SpectralGeom();
    const SpectralGeom g = best_geometry(d, w_shift, speck::matrix_form(d.Norb), spectral_layout);
    if (!g.on)
        return g;
    const double flops = direct_flops(d);
    const bool mfma = d.prec == SSE_FP32 || d.prec == SSE_BF16X3;
    const double rate = d.prec == SSE_BF16X3 ? 100e6 : d.prec == SSE_FP32 ? 50e6 : 55e6;
    const double direct = 10.0 + d.ncomp * std::max(flops / rate, 5.0 * d.NB * d.Nqz);
    return spectral_us(d, g) < direct && (!mfma || flops > 3e10) ? g : SpectralGeom();
}

SpectralGeom spectral_pi_geometry(const sse_desc &d, const int32_t *w_shift)
{
    if (d.prec != SSE_FP64)
        return SpectralGeom();
    SpectralGeom g = best_geometry(d, w_shift, speck::matrix_form(d.Norb), spectral_pi_layout);
    if (!g.on)
        return g;
    if (g.matrix) {
        // rounds of 16 points as for Sigma
        while (g.P < 64 && 2 * g.P <= g.npt && (int64_t)d.NA * g.nc * (g.npt / (2 * g.P)) >= 2048)
            g.P *= 2;
        g.npg = (g.npt + g.P - 1) / g.P;
        g.sand_lds = (size_t)speck::matrix_tiles(d.Norb) * 128 * std::min(d.NB, speck::pi_matrix_neighbours(d.Norb));
    } else
        // the sum over a point's rows reuses the Y^ region for nine values per lane
        g.sand_lds = std::max((size_t)d.Norb * d.Norb, (size_t)kNF * d.Norb) * g.P * 16 +
                 (size_t)kN3D * d.Norb * d.Norb * 8;
    // the direct kernel walks all energies of all momenta in steps of 3.2 us
    const double direct = 10.0 + d.ncomp * std::max(direct_flops(d) / 30e6, 3.2 * d.Nkz * d.NE);
    return spectral_us(d, g) < direct ? g : SpectralGeom();
}

}  // namespace sse
