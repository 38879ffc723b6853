// sse_spectral.h -- declarations of the spectral form of the self-energies: the
// (qz, w) sums of Eq. (3) are a cyclic convolution over the momenta and a linear
// one over the energies, so they are taken as products of discrete Fourier
// transforms (overlap-save blocks of L energies), all in binary64.
#pragma once

#include "sse_internal.h"

namespace sse {

namespace speck {
constexpr int kSandBlock = 256;     // threads of the sandwich kernel
constexpr int kFftBlock = 512;      // most threads of a transform kernel
constexpr size_t kLdsTwo = 79 * 1024;   // LDS of a workgroup when two share a CU
constexpr size_t kLdsOne = 158 * 1024;  // LDS of a workgroup alone on a CU
constexpr int kMaxNorb = 16;        // orbitals that the sandwich kernel is built for
constexpr size_t kAlign = 256;
// Transform lengths R1 R2 that the kernels are built for: X(R1, R2).  Close enough that
// the last energy block is rarely much larger than its energies; up to two factors that
// fit a thread's registers (18 complex values).
#define SSE_SPECTRAL_LENGTHS(X)                                                          \
    X(4, 4) X(4, 6) X(4, 8) X(6, 8) X(8, 8) X(8, 9) X(8, 10) X(8, 12) X(10, 12)          \
    X(12, 12) X(10, 16) X(12, 15) X(12, 16) X(14, 16) X(15, 16) X(16, 16) X(16, 18)
// Workspace: what a pass may hold beside its D~ and one energy block of G (soft),
// and the most a plan asks for (hard; above it the direct kernels run).
constexpr size_t kSoftBytes = (size_t)5 << 30;
constexpr size_t kHardBytes = (size_t)8 << 30;
// The matrix form of the sandwich works in tiles of four orbitals, the row form on one
// row per lane.  Measured at NA 256, NB 4, NE 270, Nkz 3 (NA 12, NE 60), us per call,
// row / matrix form: Norb 4 179 / 185 (48 / 43), 5 269 / 399, 6 374 / 403 (55 / 43),
// 7 531 / 497, 8 650 / 547, 9 892 / 1002, 10 1070 / 996 (77 / 56), 11 1485 / 1163,
// 12 1741 / 1278 (86 / 59).  Above 12 its registers spill (16: 3285 / 5011).
// Pi, both components: Norb 4 371 / 417 (50 / 45), 5 536 / 785, 6 740 / 827 (64 / 54),
// 7 1004 / 986, 8 1237 / 1101, 9 1711 / 1962, 10 2122 / 1942 (89 / 71), 11 2853 / 2262,
// 12 3386 / 2457 (95 / 78).
constexpr bool matrix_form(int No) { return No == 4 || No == 7 || No == 8 || (No >= 10 && No <= 12); }
// Tiles of 4 x 4 values of dH per neighbour in LDS; bytes per neighbour with the D^ of P
// points (Pi: without); the most neighbours that are staged at once.
constexpr int matrix_tiles(int No)
{
    const int T = (No + 3) / 4;
    return kN3D * T * T + (No % 4 == 2 ? 2 * T : 0);
}
// How far an output block may lie below its energy block's peak (SpecGuard), in powers of
// two, before the direct kernel computes it again.  Binary64 results: 6.  Flat inputs come
// to 2^-4.8 at energies that one shift alone reaches (40 taps, 16 orbital pairs) and are not
// to be computed twice; an output block at 2^-6 is off by up to 1e-14 of its norm, one at
// those energies by 5e-15 (the direct kernel: 4e-16).  Complex64 storage rounds at 2^-24;
// at 2^-20 the transforms are off by 5e-10.
// Few values are all small by chance now and then, and one tile computed again costs a
// small call as much as all of it: one orbital 20, two 10, three 8.
constexpr int guard_bits(int prec, int Norb)
{
    return prec != SSE_FP64 || Norb == 1 ? 20 : Norb == 2 ? 10 : Norb == 3 ? 8 : 6;
}
// Pi's blocks [3, 3], below the rms of their correlation.
constexpr int kPiGuardBits = 6;
constexpr size_t matrix_bytes(int No, int P) { return (size_t)matrix_tiles(No) * 128 + (size_t)kNF * P * 16; }
constexpr int matrix_neighbours(int No) { return (int)(kLdsTwo / matrix_bytes(No, 16)); }
constexpr int pi_matrix_neighbours(int No) { return (int)(kLdsTwo / (matrix_tiles(No) * 128)); }
}  // namespace speck

// Geometry and workspace layout of the spectral form of one instance.
struct SpectralGeom {
    bool on = false;
    int L = 0, r1 = 0, r2 = 0;   // energies per transform, L = r1 r2
    int V = 0, nblk = 0;         // output energies per block, blocks
    int C = 0, logC = 0;         // channels (orbital pairs of atoms) per transform workgroup
    int rowp = 0;                // LDS stride of one (momentum, channel) row, complex values
    int fft_threads = 0;
    size_t fft_lds = 0;
    int smin = 0, smax = 0;
    int npt = 0;                 // transform points per block: Nkz L
    bool matrix = false;         // which form of the sandwich
    int P = 0, npg = 0;          // points per sandwich workgroup, groups of them
    size_t sand_lds = 0;
    // one pass holds nc components, nb energy blocks, and the sandwich's output for na atoms
    int nc = 0, nb = 0, na = 0;
    size_t guard_bytes = 0;      // the guard's tables, at speck::kAlign
    size_t off_suspect = 0;      // (the second of them)
    // Sigma: D^, G^ and S^ at off_d, off_g, off_s; Pi: P^, X^ and Y^ there
    size_t off_dht = 0, off_d = 0, off_g = 0, off_s = 0, bytes = 0;
};

// Sizes, tables and workspace layout of one instance, as the kernels take them.
struct SpecParams {
    int32_t NA, NB, Norb, NN, Nkz, Nqz, NE, Nw, ncomp;
    int32_t L, V, C, logC, rowp, npt, P, npg, smin, smax, nblk;
    int32_t na_cap;             // atoms that the sandwich's output has room for
    int32_t antiherm, matrix, guard_bits;
    uint32_t guard_k;           // 2^20 log2(Nkz) / 4
    int64_t g_elems, d_elems;   // one component of G and of D~
    int64_t guard_quads;        // the guard's tables in units of 16 bytes
    int64_t off_suspect;
    int64_t off_dht, off_d, off_g, off_s;
    double alpha_re, alpha_im;
    int32_t shift[kMaxTaps];    // the caller's shifts, in frequency order
};

// What one call works on: its tensors (of the pass's first component) and workspace.
// Workspace: the non-finite flag, then
//   peaks  [ncomp][nblk][NA NN] (Pi: [ncomp][NA][NB][9]), words
//   suspect  [ncomp][NA][NE], words (Sigma)
//   dht  [NA][NB][3][n][n'] = dH[a, b, j][n'][n] (not written for the matrix form)
//   Dh   [components][NA][NB][9][npt]
//   Gh   [components][blocks][NA NN][npt]
//   Sh   [components][blocks][na_cap NN][npt]
// For Pi (G the shifted component X or the opposite one Y, Sigma the result Pi)
//   Dh   P^ [components][NA][NB][9][npt], the products summed over the energy blocks
//   Gh   X^, Sh   Y^   [components][blocks][NA NN][npt]
struct SpecPtrs {
    const int32_t *neigh;
    const double *dH;
    const void *G, *D;
    void *Sigma;
    char *ws;
};

// The part of the work that one pass does: energy blocks [blk0, blk0 + nb), atoms
// [a0, a0 + na) of the sandwich's output (components: the grid's y extent).
struct SpecPass {
    int32_t blk0, nb, a0, na;
    int32_t e_off, nrow;  // forward transforms: rows [e_off, e_off + nrow) from a block's first energy,
    int64_t src_c;        // elements from one component's input to the next,
    int64_t dst;          // and the workspace offset of the result
    int32_t c0;           // the pass's first component
};

enum SpecJobs { kDht = 1, kDhat = 2, kTransform = 4 };

struct SpecOne {
    SpecParams p;
    SpecPtrs t;
    SpecPass s;
    uint32_t *status;
    int32_t jobs;    // of k_spec_prepare
    int32_t clear;   // the job kDht also clears the status word
};

// Instances of a batch in one launch: instance i (params[i]) has workgroups
// [start[i], start[i + 1]); each is done in one pass.
struct SpecMany {
    const SpecParams *params;
    uint32_t *status;
    int32_t n;
    int32_t jobs, clear;
    int32_t start[kMaxBatch + 1];
    SpecPtrs t[kMaxBatch];
};

// The same as spectral_geometry for the phonon self-energy.
SpectralGeom spectral_pi_geometry(const sse_desc &d, const int32_t *w_shift);

// Chooses L, the channels per workgroup and the workspace; g.on says whether the
// spectral form is the better one for this problem (host, sse_geometry.hip).
SpectralGeom spectral_geometry(const sse_desc &d, const int32_t *w_shift);

SpecParams spectral_params(const sse_desc &d, const SpectralGeom &g, const int32_t *w_shift);

// Sigma of every component (sse_spectral.hip), then the direct kernel (redo: its
// sizes and taps) where the non-finite flag or the guard asks for it.  clear: the status word
// first; in the end it goes to *host (pinned memory, or NULL).  Weak: a build of the host runtime alone (its CPU test)
// has no kernels to launch, and runs the direct launchers.
__attribute__((weak)) hipError_t spectral_sigma_launch(const sse_desc &d, const SpectralGeom &g,
                                                       const int32_t *w_shift, const sse_args &a,
                                                       uint32_t *status, bool clear,
                                                       uint32_t *host, const Fp64Params &redo, size_t redo_lds,
                                                       void *ws, hipStream_t s);

// The instances of a batch that one pass each can do, together: geom[i], args and
// workspace offset of each; hp are their parameters, params and redo device tables of
// the same n instances.  clear: the status word first.
__attribute__((weak)) hipError_t spectral_batch_launch(int n, const sse_desc *const *d,
                                                       const SpectralGeom *const *g, const sse_args *const *a,
                                                       const size_t *ws_off, const SpecParams *hp,
                                                       const SpecParams *params,
                                                       const Fp64Params *redo, size_t redo_lds,
                                                       uint32_t *status, bool clear, char *ws,
                                                       hipStream_t s);

// Pi of every component; the non-finite flag for the direct kernel is at the start of ws,
// the guard's tables are at speck::kAlign.
__attribute__((weak)) hipError_t spectral_pi_launch(const sse_desc &d, const SpectralGeom &g,
                                                    const int32_t *w_shift, const int32_t *neigh, const double *dH,
                                                    const void *G, void *Pi, uint32_t *status, void *ws,
                                                    hipStream_t s);

}  // namespace sse
