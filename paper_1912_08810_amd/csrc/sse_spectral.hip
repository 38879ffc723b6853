// sse_spectral.hip -- the self-energies in the transform domain, binary64.
//
// Eq. (3) (Sec. 2) sums over q cyclically in k and over the shifts s_w in e:
//   Sigma[k, e, a] = alpha sum_b sum_ij dH_i . ( sum_q sum_w Dt_ij[q, w, a, b]
//                                              G[(k - q) mod Nkz, e - s_w, f] ) . dH_j^T
// so a discrete Fourier transform over k (length Nkz) and over energy blocks
// (length L) turns the (q, w) sums into one product per transform point
// (kappa, eps); dH does not depend on k or e, so it stays outside:
//   S^[kappa, eps, a] = sum_b sum_ij D^_ij[kappa, eps, a, b] dH_i . G^[kappa, eps, f] . dH_j^T
// Overlap-save: block n holds the G rows e0 - smax + r, r < L, of its V = L -
// (smax - smin) output energies e0 + v; with t_w = smax - s_w,
//   y[v] = sum_w D_w x[v + t_w],  y^[eps] = x^[eps] sum_w D_w exp(+2 pi i eps t_w / L).
// The tap sums cost 72 Nqz Nw flops per (k, e, a, b, orbital pair) in the direct
// kernels and 72 here, next to 24 Norb for the dH products.
//
// Passes (each one launch over the pass's components and energy blocks):
//   k_spec_prepare   up to three independent jobs by workgroup: dH transposed for
//                    scalar reads (and the status word and flag cleared), D^, G -> G^
//   k_spec_sandwich  G^, D^ -> S^ (for the Norb that speck::matrix_form names
//                    k_spec_matrix, and k_spec_pi_matrix in place of k_spec_pi)
//   k_spec_inverse   S^ -> Sigma, and the neighbour-table check
//   k_sse_fp64_redo  the direct kernel: all of it, or what the guard has marked
// Twiddle factors are computed by each workgroup into LDS, so that nothing has to run
// before the first launch.
// G^ and S^ are laid out [atom, orbital pair][kappa][eps], points fastest, so every
// pass reads and writes whole runs of points.  Rounding is that of binary64
// transforms: relative to the largest values of an energy block; outputs that lie far
// below it are computed again by the direct kernel (SpecGuard).
// Device scale (NA = 1024, NB = 4, Norb = 10, Nkz = Nqz = 7, NE = 1000, Nw = 30, both
// components, complex128): 1609 ms per call in the direct kernel, 73 ms here: the sandwich
// 47 ms, k_spec_prepare 14.4 (3.9 TB/s), k_spec_inverse 11.5 (4.5 TB/s).
// Inputs that are not finite, or so large that a transform overflows, raise a flag;
// the direct kernel then recomputes Sigma (its sums meet fewer elements).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstring>

#include "sse_copy.h"
#include "sse_dft.h"
#include "sse_guard.h"
#include "sse_spectral.h"

namespace sse {

namespace {

constexpr int kSB = speck::kSandBlock;

__device__ __forceinline__ int64_t xcd_remap(int64_t bid, int64_t n)
{
    const int64_t per = n >> 3;
    if (bid >= (per << 3))
        return bid;
    return (bid & 7) * per + (bid >> 3);
}

__device__ __forceinline__ double2 to_d2(double2 v) { return v; }
__device__ __forceinline__ double2 to_d2(float2 v) { return make_double2(v.x, v.y); }
__device__ __forceinline__ void put(double2 *p, double x, double y) { *p = make_double2(x, y); }
__device__ __forceinline__ void put(float2 *p, double x, double y) { *p = make_float2((float)x, (float)y); }

// Whether transforms of values like x stay finite: sums of up to 2^15 of them.
__device__ __forceinline__ bool finite(double x) { return __builtin_fabs(x) <= 0x1p1000; }

// A workgroup's instance, pass and index in it.
struct Job {
    const_ptr<SpecParams> p;
    SpecPtrs t;
    SpecPass s;
    int64_t bid;

    __device__ __forceinline__ uint32_t *flag() const { return reinterpret_cast<uint32_t *>(t.ws); }
    __device__ __forceinline__ uint32_t *peaks() const { return reinterpret_cast<uint32_t *>(t.ws + speck::kAlign); }
    __device__ __forceinline__ uint32_t *suspect() const { return reinterpret_cast<uint32_t *>(t.ws + p->off_suspect); }
    __device__ __forceinline__ double *dht() const { return reinterpret_cast<double *>(t.ws + p->off_dht); }
    __device__ __forceinline__ double2 *Dh() const { return reinterpret_cast<double2 *>(t.ws + p->off_d); }
    __device__ __forceinline__ double2 *Gh() const { return reinterpret_cast<double2 *>(t.ws + p->off_g); }
    __device__ __forceinline__ double2 *Sh() const { return reinterpret_cast<double2 *>(t.ws + p->off_s); }
};
__device__ __forceinline__ Job job(const SpecOne &o)
{
    return Job{ro(&o.p), o.t, o.s, blockIdx.x};
}
__device__ __forceinline__ Job job(const SpecMany &m)
{
    int lo = 0, hi = m.n - 1;
    const int x = blockIdx.x;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (m.start[mid] <= x)
            lo = mid;
        else
            hi = mid - 1;
    }
    lo = __builtin_amdgcn_readfirstlane(lo);
    const_ptr<SpecParams> p = ro(m.params) + lo;
    return Job{p, m.t[lo], SpecPass{0, p->nblk, 0, p->NA, -p->smax, p->L, p->g_elems, p->off_g}, x - m.start[lo]};
}

// tw[j] = exp(-2 pi i j m / n) for j < count.
__device__ __forceinline__ void fill_twiddles(double2 *tw, int count, int m, int n)
{
    for (int i = threadIdx.x; i < count; i += blockDim.x) {
        int j = (int)((int64_t)i * m % n);
        if (2 * j > n)  // the angle in (-1, 1] half turns
            j -= n;
        double s, c;
        sincospi(2.0 * j / n, &s, &c);
        tw[i] = make_double2(c, -s);
    }
}

constexpr int kPlainAtoms = 256;

// Workgroups of one instance in each job.
__host__ __device__ inline int64_t dht_wgs(const SpecParams &p)
{
    const int64_t d = p.matrix ? 0 : (int64_t)p.NA * p.NB * kN3D * p.NN;
    const int64_t n = ((d > p.guard_quads ? d : p.guard_quads) + 1023) / 1024;
    return n < 512 ? n : 512;
}
__host__ __device__ inline int64_t dhat_wgs(const SpecParams &p) { return (int64_t)p.NA * p.NB * p.Nkz; }
__host__ __device__ inline int64_t fft_wgs(const SpecParams &p, int64_t atoms, int nb)
{
    return ((atoms * p.NN + p.C - 1) >> p.logC) * nb;
}
// Groups of channels of the inverse transforms: where an atom has more than C, of one atom
// each (nearly as many in each of them), so that the guard meets no half ones.
__host__ __device__ inline int64_t inverse_groups(const SpecParams &p, int64_t atoms)
{
    return p.NN > p.C ? atoms * ((p.NN + p.C - 1) >> p.logC) : (atoms * p.NN + p.C - 1) >> p.logC;
}
__host__ __device__ inline int64_t sandwich_wgs(const SpecParams &p, int na, int nb)
{
    return (int64_t)(na < kPlainAtoms ? na : (na + 7) / 8 * 8) * p.npg * nb;
}
// The atom of a sandwich workgroup and its point group (counted over the energy blocks);
// false: none.  All XCDs work on one group of points at a time (its G^ rows stay in the
// last-level cache), an XCD on neighbouring atoms.  With few atoms, whose eighths would
// differ (12 atoms: two XCDs idle), they are dealt out one by one: a batch of 8 to 16
// atoms each 372 -> 334 us, 97 atoms 737 -> 703 us.  One by one and in eighths, us per
// component (Norb 10, NB 4, NE 270, Nkz 3): 64 atoms 204 and 211, 128 387 and 382, 256 710
// and 708, 512 1359 and 1352, 1024 2604 and 2575.
__device__ __forceinline__ bool sandwich_place(int64_t bid, int na, int64_t groups, int *atom, int64_t *group)
{
    if (na < kPlainAtoms) {
        *atom = (int)(bid % na);
        *group = bid / na;
    } else {
        const int na8 = (na + 7) >> 3, per = na8 * 8, in = (int)(bid % per);
        *atom = (in & 7) * na8 + (in >> 3);
        *group = bid / per;
    }
    return *atom < na && *group < groups;
}

// dH^T, and the flag, the guard's tables (and the status word) cleared; workgroup bid of nwg.
__device__ __forceinline__ void dht_job(const Job &J, int64_t bid, int64_t nwg, uint32_t *clear)
{
    const auto &p = *J.p;
    const int64_t i0 = bid * blockDim.x + threadIdx.x, step = nwg * blockDim.x;
    if (i0 == 0) {
        *J.flag() = 0u;
        if (clear)
            *clear = 0u;
    }
    uint4 *guard = reinterpret_cast<uint4 *>(J.peaks());
    for (int64_t i = i0; i < p.guard_quads; i += step)
        guard[i] = make_uint4(0u, 0u, 0u, 0u);
    if (p.matrix)
        return;
    double *dht = J.dht();
    const int NN = p.NN, No = p.Norb;
    const int64_t nd = (int64_t)p.NA * p.NB * kN3D * NN;
    for (int64_t i = i0; i < nd; i += step) {
        const int64_t blk = i / NN;
        const int c = (int)(i - blk * NN), n = c / No, np = c - n * No;
        dht[i] = J.t.dH[blk * NN + np * No + n];
    }
}

// D^_ij[kappa, eps] of one (a, b) and kappa: the q sum into LDS (a few kB), then each
// thread takes an eps and all nine (i, j).
template <typename T>
__device__ __forceinline__ void dhat_job(const Job &J, double2 *lds, int64_t bid)
{
    const auto &p = *J.p;
    const int64_t ab = bid / p.Nkz;
    const int kap = (int)(bid - ab * p.Nkz), tid = threadIdx.x;
    double2 *tw = lds;               // [L]
    double2 *tq = tw + p.L;          // [Nqz]
    double2 *Dk = tq + p.Nqz;        // [Nw][9]
    const T *D = (const T *)J.t.D + (size_t)blockIdx.y * p.d_elems;
    const int64_t slab = (int64_t)p.NA * p.NB * kNF;
    fill_twiddles(tw, p.L, 1, p.L);
    fill_twiddles(tq, p.Nqz, kap, p.Nkz);
    __syncthreads();
    for (int i = tid; i < p.Nw * kNF; i += blockDim.x) {
        const int w = i / kNF, ij = i - w * kNF;
        // an anti-Hermitian D~ is completed from its entries i < j and Im of the diagonal
        const int ii = ij / kN3D, jj = ij - ii * kN3D;
        const bool low = p.antiherm && ii > jj, dia = p.antiherm && ii == jj;
        const T *src = D + ((int64_t)w * slab + ab * kNF + (low ? jj * kN3D + ii : ij));
        double xr = 0.0, xi = 0.0;
#pragma unroll 4
        for (int q = 0; q < p.Nqz; ++q) {
            double2 v = to_d2(src[(int64_t)q * p.Nw * slab]);
            if (low || dia)
                v.x = dia ? 0.0 : -v.x;
            const double2 t = tq[q];
            xr = fma(v.x, t.x, fma(-v.y, t.y, xr));
            xi = fma(v.x, t.y, fma(v.y, t.x, xi));
        }
        Dk[i] = make_double2(xr, xi);
    }
    __syncthreads();
    double2 *out = J.Dh() + ((size_t)blockIdx.y * p.NA * p.NB + ab) * kNF * p.npt + (size_t)kap * p.L;
    for (int e = tid; e < p.L; e += blockDim.x) {
        double ar[kNF], ai[kNF];
#pragma unroll
        for (int x = 0; x < kNF; ++x)
            ar[x] = ai[x] = 0.0;
        for (int w = 0; w < p.Nw; ++w) {
            const double2 t = tw[e * (p.smax - p.shift[w]) % p.L];  // conjugated below
#pragma unroll
            for (int x = 0; x < kNF; ++x) {
                const double2 d = Dk[w * kNF + x];
                ar[x] = fma(d.x, t.x, fma(d.y, t.y, ar[x]));
                ai[x] = fma(d.y, t.x, fma(-d.x, t.y, ai[x]));
            }
        }
#pragma unroll
        for (int x = 0; x < kNF; ++x)
            out[(size_t)x * p.npt + e] = make_double2(ar[x], ai[x]);
    }
}

// f over 2^lw lanes side by side, in all of them.
template <typename F>
__device__ __forceinline__ uint32_t over_lanes(uint32_t x, int lw, F f)
{
    if (lw > 0)
        x = f(x, (uint32_t)__builtin_amdgcn_mov_dpp((int)x, 0xB1, 0xf, 0xf, true));   // lane ^ 1
    if (lw > 1)
        x = f(x, (uint32_t)__builtin_amdgcn_mov_dpp((int)x, 0x4E, 0xf, 0xf, true));   // lane ^ 2
    if (lw > 2)
        x = f(x, (uint32_t)__builtin_amdgcn_mov_dpp((int)x, 0x141, 0xf, 0xf, true));  // lane ^ 7
    return x;
}

// The largest value of a channel's rows in LDS: in the padding of the channel's first row.
template <int R2>
__device__ __forceinline__ uint32_t *channel_top(double2 *lds, int ch, int rowp)
{
    return reinterpret_cast<uint32_t *>(lds + (size_t)ch * rowp + R2);
}

// The middle step of a transform of length R1 R2 in LDS: the R2-point transforms.  Peak: the
// channels' largest values (row r: channel r & mask) go where channel_top says.
template <int R1, int R2, int S, bool Peak>
__device__ __forceinline__ void second_step(double2 *lds, int rows, int rowp, int mask)
{
    for (int it = threadIdx.x; it < rows * R1; it += blockDim.x) {
        const int row = it / R1, k1 = it - row * R1;
        double2 *x = lds + (size_t)row * rowp + k1 * (R2 + 1);
        double2 v[R2];
#pragma unroll
        for (int n = 0; n < R2; ++n)
            v[n] = x[n];
        dft::transform<R2, S>(v);
        double most = 0.0;
#pragma unroll
        for (int n = 0; n < R2; ++n) {
            x[n] = v[n];
            if (Peak)
                most = fmax(most, fmax(fabs(v[n].x), fabs(v[n].y)));
        }
        if (Peak) {
            // lanes side by side have the same row
            constexpr int lw = R1 % 4 == 0 ? 2 : R1 % 2 == 0 ? 1 : 0;
            const uint32_t top = over_lanes(magnitude(most), lw, [](uint32_t a, uint32_t b) { return max(a, b); });
            if ((threadIdx.x & ((1 << lw) - 1)) == 0)
                atomicMax(channel_top<R2>(lds, row & mask, rowp), top);
        }
    }
}

// The transform over the momenta of the N values at y (stride values apart): put(k, value).
template <int N, int S, typename Put>
__device__ __forceinline__ void k_transform_as(const double2 *y, size_t stride, Put put)
{
    double2 v[N];
#pragma unroll
    for (int k = 0; k < N; ++k)
        v[k] = y[k * stride];
    dft::transform<N, S>(v);
#pragma unroll
    for (int k = 0; k < N; ++k)
        put(k, v[k]);
}
template <int S, typename Put>
__device__ __forceinline__ void k_transform(int Nkz, const double2 *y, size_t stride, const double2 *twk, Put put)
{
    switch (Nkz) {
    case 1: return k_transform_as<1, S>(y, stride, put);
    case 2: return k_transform_as<2, S>(y, stride, put);
    case 3: return k_transform_as<3, S>(y, stride, put);
    case 4: return k_transform_as<4, S>(y, stride, put);
    case 5: return k_transform_as<5, S>(y, stride, put);
    case 6: return k_transform_as<6, S>(y, stride, put);
    case 7: return k_transform_as<7, S>(y, stride, put);
    case 8: return k_transform_as<8, S>(y, stride, put);
    }
    for (int kap = 0; kap < Nkz; ++kap) {
        double xr = 0.0, xi = 0.0;
        int j = 0;
        for (int k = 0; k < Nkz; ++k) {
            const double2 v = y[k * stride], t = twk[j];
            xr = fma(v.x, t.x, fma(S * v.y, t.y, xr));
            xi = fma(-S * v.x, t.y, fma(v.y, t.x, xi));
            j += kap;
            j -= j >= Nkz ? Nkz : 0;
        }
        put(kap, make_double2(xr, xi));
    }
}

// Transform size L = R1 R2 as n = R2 n1 + n2, eps = k1 + R1 k2: R1-point transforms
// straight from global memory (R1 loads in flight per thread), twiddles, R2-point
// transforms in LDS, then the transform over k on the way out.  A workgroup takes C
// consecutive channels (64-byte pieces of each energy row) and all Nkz momenta.
// S is the sign of the exponents: -1, or +1 for the opposite component of the phonon
// self-energy, whose transform is wanted at the negated point.
// LDS: [L] and [Nkz] twiddle factors, then the rows [Nkz][C].
template <typename T, int R1, int R2, int S>
__device__ __forceinline__ void forward_job(const Job &J, const SpecPass &s, double2 *lds, int64_t bid)
{
    constexpr int L = R1 * R2;
    const auto &p = *J.p;
    const int C = p.C, NC = p.NA * p.NN, Nkz = p.Nkz, rowp = p.rowp;
    const int ngrp = (NC + C - 1) >> p.logC;
    if (bid >= (int64_t)ngrp * s.nb)
        return;
    const int64_t x = xcd_remap(bid, (int64_t)ngrp * s.nb);
    const int blk = (int)(x / ngrp), ch0 = (int)(x - (int64_t)blk * ngrp) << p.logC;
    const T *src = (const T *)J.t.G + (int64_t)blockIdx.y * s.src_c;
    double2 *tw = lds, *twk = lds + L;
    lds += L + Nkz;
    const int ebase = (s.blk0 + blk) * p.V + s.e_off, nrow = s.nrow, items = Nkz * C * R2;
    double2 v[R1];
    auto load = [&](int it) {
        const int ch = it & (C - 1), r = it >> p.logC, k = r / R2, n2 = r - k * R2;
        const bool ok = ch0 + ch < NC;
        const T *row = src + (int64_t)k * p.NE * NC + ch0 + ch;
#pragma unroll
        for (int n1 = 0; n1 < R1; ++n1) {
            const int rr = n1 * R2 + n2, e = ebase + rr;
            v[n1] = ok && rr < nrow && e >= 0 && e < p.NE ? to_d2(row[(int64_t)e * NC]) : make_double2(0.0, 0.0);
        }
    };
    // the first loads are under way while the twiddles are computed (one GPU's energy
    // shard 13.1 -> 12.7 ms, a batch of tiny instances 334 -> 325 us, here and in inverse_job)
    int it = threadIdx.x;
    if (it < items)
        load(it);
    fill_twiddles(tw, L, 1, L);
    fill_twiddles(twk, Nkz, 1, Nkz);
    __syncthreads();
    while (it < items) {
        const int ch = it & (C - 1), r = it >> p.logC, k = r / R2, n2 = r - k * R2;
        dft::transform<R1, S>(v);
        double2 *o = lds + (size_t)(k * C + ch) * rowp + n2;
        o[0] = v[0];
#pragma unroll
        for (int k1 = 1; k1 < R1; ++k1) {
            const double2 t = tw[k1 * n2];
            o[k1 * (R2 + 1)] = dft::cmul(v[k1], t.x, -S * t.y);
        }
        it += blockDim.x;
        if (it < items)
            load(it);
    }
    __syncthreads();
    second_step<R1, R2, S, false>(lds, Nkz * C, rowp, 0);
    __syncthreads();
    double2 *out = reinterpret_cast<double2 *>(J.t.ws + s.dst) + (((size_t)blockIdx.y * s.nb + blk) * NC + ch0) * p.npt;
    for (int it = threadIdx.x; it < L * C; it += blockDim.x) {
        const int ch = it / L, eps = it - ch * L;
        if (ch0 + ch >= NC)
            break;
        const double2 *y = lds + (size_t)ch * rowp + (eps % R1) * (R2 + 1) + eps / R1;
        double2 *o = out + (size_t)ch * p.npt + eps;
        k_transform<S>(Nkz, y, (size_t)C * rowp, twk, [&](int kap, double2 v) { o[(size_t)kap * L] = v; });
    }
}

// The same backwards: energies from points, then k on the way out, alpha and 1 / (Nkz L).
// An energy that no shift reaches gets an exact zero, as the direct sum gives.  Also
// the neighbour-table check.
// The guard (SpecGuard): a channel's peak is the largest value before the transform over k,
// the discarded energies' among them, times Nkz^(1/4): the rounding is relative to the root
// of the sum of the squares over kappa, between one and Nkz^(1/2) times that.  An atom's peak
// is its channels' largest.  Where the outputs of a few of its channels lie below those
// channels' own peak, the atom's output is marked as suspect; where no such few do, all its
// channels together do not lie below the atom's.  The direct kernel looks at what is marked
// (of flat inputs one in 1e10, and some at energies that few shifts reach).  One GPU's energy
// shard: 935 us per component without it, 980 with it (the largest value of every output in a
// table, by atomics from the channels' workgroups: 1124); a batch of tiny instances 45 and
// 55 us, 256 atoms in complex64 280 and 307.
template <typename T, int R1, int R2>
__device__ __forceinline__ void inverse_job(const Job &J, double2 *lds, uint32_t *status)
{
    constexpr int L = R1 * R2;
    const auto &p = *J.p;
    const int C = p.C, Nkz = p.Nkz, rowp = p.rowp;
    const int64_t strideE = (int64_t)p.NA * p.NN;
    const int ngrp = (int)inverse_groups(p, J.s.na);
    if (J.bid >= (int64_t)ngrp * J.s.nb)
        return;
    const int64_t x = xcd_remap(J.bid, (int64_t)ngrp * J.s.nb);
    const int blk = (int)(x / ngrp), grp = (int)(x - (int64_t)blk * ngrp);
    // channels [ch0, NC) of the group, at most C
    int ch0 = grp << p.logC, NC = min(ch0 + C, J.s.na * p.NN);
    if (p.NN > C) {
        const int per = (p.NN + C - 1) >> p.logC, al = grp / per, i = grp - al * per;
        ch0 = al * p.NN + i * p.NN / per;
        NC = al * p.NN + (i + 1) * p.NN / per;
    }
    const int64_t nab = (int64_t)p.NA * p.NB, all = (int64_t)ngrp * J.s.nb * blockDim.x;
    if (blockIdx.y == 0)
        for (int64_t i = J.bid * blockDim.x + threadIdx.x; i < nab; i += all)
            if ((unsigned)J.t.neigh[i] >= (unsigned)p.NA)
                atomicOr(status, kStatusBadNeigh);
    const double2 *src = J.Sh() + (((size_t)blockIdx.y * J.s.nb + blk) * p.na_cap * p.NN + ch0) * p.npt;
    double2 *tw = lds, *twk = lds + L;
    lds += L + Nkz;
    const int items = Nkz * C * R2;
    double2 v[R1];
    auto load = [&](int it) {
        const int row = it / R2, n2 = it - row * R2, ch = row & (C - 1), kap = row >> p.logC;
        const bool ok = ch0 + ch < NC;
        const double2 *y = src + (size_t)ch * p.npt + kap * L + n2;
#pragma unroll
        for (int n1 = 0; n1 < R1; ++n1)
            v[n1] = ok ? y[n1 * R2] : make_double2(0.0, 0.0);
    };
    int it = threadIdx.x;
    if (it < items)
        load(it);
    if (threadIdx.x < C)
        *channel_top<R2>(lds, threadIdx.x, rowp) = 0u;
    fill_twiddles(tw, L, 1, L);
    fill_twiddles(twk, Nkz, 1, Nkz);
    __syncthreads();
    while (it < items) {
        const int row = it / R2, n2 = it - row * R2;
        dft::transform<R1, 1>(v);
        double2 *o = lds + (size_t)row * rowp + n2;
        o[0] = v[0];
#pragma unroll
        for (int k1 = 1; k1 < R1; ++k1) {
            const double2 t = tw[k1 * n2];
            o[k1 * (R2 + 1)] = dft::cmul(v[k1], t.x, -t.y);
        }
        it += blockDim.x;
        if (it < items)
            load(it);
    }
    __syncthreads();
    second_step<R1, R2, 1, true>(lds, Nkz * C, rowp, C - 1);
    __syncthreads();
    const double sc = 1.0 / ((double)Nkz * L);
    const double ar = p.alpha_re * sc, ai = p.alpha_im * sc;
    const int e0 = (J.s.blk0 + blk) * p.V, nv = min(p.V, p.NE - e0);
    T *dst = (T *)J.t.Sigma + (size_t)blockIdx.y * p.g_elems + (size_t)J.s.a0 * p.NN + ch0;
    // A lane keeps its channel: the workgroup has a multiple of C threads.  2^lw channels of
    // one atom side by side are the few: all of the group's, or (C of several atoms) an atom's.
    // Lanes past the last channel repeat it.
    const int ch = min((int)(threadIdx.x & (C - 1)), NC - 1 - ch0);
    const int lw = p.NN > C ? p.logC : __builtin_ctz(p.NN);
    const uint32_t peak = over_lanes(*channel_top<R2>(lds, ch, rowp) + p.guard_k, lw,
                                     [](uint32_t x, uint32_t y) { return max(x, y); });
    const uint32_t least = guard_floor(peak, p.guard_bits);
    const int64_t comp = J.s.c0 + blockIdx.y;
    if (threadIdx.x < C)
        J.peaks()[(comp * p.nblk + J.s.blk0 + blk) * strideE + J.s.a0 * p.NN + ch0 + ch] = peak;
    // low: a bit per momentum, whether the value lies below least; of the few together
    auto together = [&](uint32_t low) { return over_lanes(low, lw, [](uint32_t x, uint32_t y) { return x & y; }); };
    bool marked = false;
    for (int it = threadIdx.x; it < nv * C; it += blockDim.x) {
        const int vv = it >> p.logC, e = e0 + vv;
        bool reached = false;
        for (int w = 0; w < p.Nw && !reached; ++w)
            reached = e - p.shift[w] >= 0 && e - p.shift[w] < p.NE;
        uint32_t low = 0u, any = 0u;
        const double2 *y = lds + (size_t)ch * rowp + (vv % R1) * (R2 + 1) + vv / R1;
        T *o = dst + (int64_t)e * strideE + ch;
        k_transform<1>(Nkz, y, (size_t)C * rowp, twk, [&](int k, double2 s) {
            low = low + low + (magnitude(s) < least ? 1u : 0u);
            if ((k & 31) == 31)
                any |= together(low);
            if (reached)
                put(o + (int64_t)k * p.NE * strideE, ar * s.x - ai * s.y, ar * s.y + ai * s.x);
            else
                put(o + (int64_t)k * p.NE * strideE, 0.0, 0.0);
        });
        any |= together(low);
        marked |= any && reached;
        if (any && reached)
            atomicOr(&J.suspect()[(comp * p.NA + J.s.a0 + (ch0 + ch) / p.NN) * p.NE + e], any);
    }
    if (__any(marked) && (threadIdx.x & 63) == 0)
        atomicOr(J.flag(), kFlagSuspect);
}

// Calls f with the integral constants R1, R2 of the transform length L.
template <typename F>
__host__ __device__ __forceinline__ void with_length(int L, F f)
{
    using std::integral_constant;
    switch (L) {
#define SSE_LENGTH(R1, R2)                                                     \
    case R1 * R2:                                                              \
        f(integral_constant<int, R1>{}, integral_constant<int, R2>{});         \
        break;
        SSE_SPECTRAL_LENGTHS(SSE_LENGTH)
#undef SSE_LENGTH
    }
}

// The jobs before the sandwich, as many of them as arg.jobs names: in one launch for
// small problems, which wait for launches; D^ apart from the transforms for others,
// whose LDS would leave its workgroups alone on a CU (one GPU's energy shard: 2.37 ms
// together, 1.77 ms apart).  R1 = 0: the length is the instance's own (a batch).
template <typename T, int R1, int R2, typename A>
__global__ __launch_bounds__(speck::kFftBlock, 4) void k_spec_prepare(const A arg)
{
    extern __shared__ double2 lds[];
    const Job J = job(arg);
    const SpecParams &p = *(const SpecParams *)J.p;
    const int64_t n0 = arg.jobs & kDht ? dht_wgs(p) : 0, n1 = n0 + (arg.jobs & kDhat ? dhat_wgs(p) : 0);
    if (J.bid < n0) {
        if (blockIdx.y == 0)
            dht_job(J, J.bid, n0, arg.clear ? arg.status : nullptr);
    } else if (J.bid < n1) {
        dhat_job<T>(J, lds, J.bid - n0);
    } else if constexpr (R1 > 0) {
        forward_job<T, R1, R2, -1>(J, J.s, lds, J.bid - n1);
    } else {
        with_length(p.L, [&](auto r1, auto r2) {
            forward_job<T, decltype(r1)::value, decltype(r2)::value, -1>(J, J.s, lds, J.bid - n1);
        });
    }
}

template <typename T, int R1, int R2, typename A>
__global__ __launch_bounds__(speck::kFftBlock, 4) void k_spec_inverse(const A arg)
{
    extern __shared__ double2 lds[];
    const Job J = job(arg);
    if constexpr (R1 > 0)
        inverse_job<T, R1, R2>(J, lds, arg.status);
    else
        with_length(J.p->L, [&](auto r1, auto r2) {
            inverse_job<T, decltype(r1)::value, decltype(r2)::value>(J, lds, arg.status);
        });
}

// The jobs before k_spec_pi: dH^T (first pass), then X^ and Y^ of the pass's energy blocks.
template <int R1, int R2>
__global__ __launch_bounds__(speck::kFftBlock, 4) void k_spec_pi_prepare(const SpecOne arg)
{
    extern __shared__ double2 lds[];
    Job J = job(arg);
    const SpecParams &p = *(const SpecParams *)J.p;
    const int64_t n0 = arg.jobs & kDht ? dht_wgs(p) : 0, nf = fft_wgs(p, p.NA, J.s.nb);
    SpecPass s = J.s;
    if (J.bid < n0) {
        if (blockIdx.y == 0)
            dht_job(J, J.bid, n0, arg.status);
    } else if (J.bid < n0 + nf) {
        s.e_off = p.smin;
        s.nrow = p.L;
        s.src_c = p.g_elems;
        s.dst = p.off_g;
        forward_job<double2, R1, R2, -1>(J, s, lds, J.bid - n0);
    } else {
        J.t.G = J.t.D;  // the opposite component
        s.e_off = 0;
        s.nrow = p.V;
        s.src_c = -p.g_elems;
        s.dst = p.off_s;
        forward_job<double2, R1, R2, 1>(J, s, lds, J.bid - n0 - nf);
    }
}

// Keeps a value's computation where it stands: the compiler would otherwise sink the
// FMAs of a loop past the branches that follow it, holding every operand meanwhile.
__device__ __forceinline__ void pin(double &x) { asm volatile("" : "+v"(x)); }

// S^[a][m, n'][point] = sum_b sum_ij D^_ij[point] (dH_i . G^_f[point] . dH_j^T)[m][n'].
// A workgroup takes P points of one atom; a lane takes row m of one point.  Per
// neighbour and block of CB columns it forms M_i[m, n] = (dH_i G^)[m, n] from LDS, then
// T_j[m, n] = sum_i D^_ij M_i[m, n] and adds T_j[m, n] dH_j[:, n] to its row of S^ with the
// wave-uniform dH_j in scalar registers.  Both halves are pipelined by hand (the
// compiler waits for every read where it is used): kAhead LDS reads are in flight
// ahead of the FMAs that need them, and the scalar loads of step (j, n + 1) during
// step (j, n), one wait per step (scalar loads complete out of order, so a wait for
// one is a wait for all).  The next neighbour's G^ is copied into LDS during the
// second half, which does not read it.
//
// Bound: binary64 FMA issue, and the power it takes.  NA 256, NB 4, NE 270, Nkz 3, per
// component: Norb 9 626 us, 16 2.51 ms.  The vector units are busy 75 and 70 % of the
// cycles, 86 and 88 % of the vector instructions are FMAs (1440 per lane and neighbour at
// Norb 9), and the clock sinks from 2.4 to 1.8 GHz (FMA issue at 2.4 GHz: 297 us and
// 1.31 ms).  Before the hand pipelining it took twice as long; leaving out the copies, the
// scalar loads or the LDS reads shortens it by 8 to 14 % each (both seen at Norb 10): none of
// them alone is what it waits for.
template <int No, int CB, int W, typename A>
__global__ __launch_bounds__(kSB, W) void k_spec_sandwich(const A arg)
{
    extern __shared__ double2 lds[];
    const Job J = job(arg);
    const auto &p = *J.p;
    constexpr int kAhead = CB < 4 ? CB : 4;  // at most a row: h holds two
    constexpr int NN = No * No, P = kSB / No;
    constexpr int NC = (No + CB - 1) / CB;                  // column blocks; the last may be ragged
    double *hs = reinterpret_cast<double *>(lds + NN * P);  // [3][No][No]
    int al;
    int64_t x;
    if (!sandwich_place(J.bid, J.s.na, (int64_t)p.npg * J.s.nb, &al, &x))
        return;
    const int pg = (int)(x % p.npg), blk = (int)(x / p.npg);
    const int a = J.s.a0 + al, pt0 = pg * P, npt = p.npt;
    const int tid = threadIdx.x, m = tid / P, pt = tid - m * P;
    const bool act = m < No && pt0 + pt < npt;
    const int mr = act ? m : 0, pr = act ? pt : 0;
    const double2 *Gh = J.Gh() + ((size_t)blockIdx.y * J.s.nb + blk) * p.NA * NN * npt + pt0;
    const double2 *Dh = J.Dh() + ((size_t)blockIdx.y * p.NA + a) * p.NB * kNF * npt + pt0;
    const int np = min(P, npt - pt0);
    const_ptr<int32_t> neigh = ro(J.t.neigh) + (size_t)a * p.NB;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);

    auto next_valid = [&](int b) {
        while (b < p.NB && (unsigned)neigh[b] >= (unsigned)p.NA)
            ++b;
        return b;
    };
    // start the copies of neighbour b's G^ points (those past the last point repeat it)
    // and dH into LDS; 32-bit offsets from uniform bases
    auto issue = [&](int b) {
        int t = tid;
        asm volatile("" : "+v"(t));  // recomputed per neighbour rather than held
        const char *g = reinterpret_cast<const char *>(Gh + (size_t)neigh[b] * NN * npt);
        uint32_t *dst = reinterpret_cast<uint32_t *>(lds) + wave * 64 * 4;
#pragma unroll
        for (int i = 0; i < (NN * P + kSB - 1) / kSB; ++i) {
            const int u = t + i * kSB, c = u / P, q = min(u - c * P, np - 1);
            if (NN * P % kSB == 0 || u < NN * P)
                lds_copy<4>(g + (unsigned)((c * npt + q) * 16), dst + i * kSB * 4);
        }
        const char *h = reinterpret_cast<const char *>(J.t.dH + ((size_t)a * p.NB + b) * kN3D * NN);
        uint32_t *hd = reinterpret_cast<uint32_t *>(hs) + wave * 64;
#pragma unroll
        for (int i = 0; i < (kN3D * NN * 2 + kSB - 1) / kSB; ++i)
            if (t + i * kSB < kN3D * NN * 2)
                lds_copy<1>(h + (unsigned)((t + i * kSB) * 4), hd + i * kSB);
    };

    double sr[No], si[No];
#pragma unroll
    for (int n = 0; n < No; ++n)
        sr[n] = si[n] = 0.0;
    int b = next_valid(0);
    if (b < p.NB)
        issue(b);
    while (b < p.NB) {
        const int bn = next_valid(b + 1);
        __syncthreads();  // neighbour b has landed
        const_ptr<double> ht = ro(J.dht() + ((size_t)a * p.NB + b) * kN3D * NN);
        const double2 *db = Dh + (size_t)b * kNF * npt;
#pragma unroll 1
        for (int cb = 0; cb < NC; ++cb) {
            const int c0 = cb * CB;
            double2 d[kN3D];  // D^_ij of the current j
#pragma unroll
            for (int i = 0; i < kN3D; ++i)
                d[i] = (db + (size_t)i * kN3D * npt)[pr];
            double xr[kN3D][CB], xi[kN3D][CB];
#pragma unroll
            for (int i = 0; i < kN3D; ++i)
#pragma unroll
                for (int n = 0; n < CB; ++n)
                    xr[i][n] = xi[i][n] = 0.0;
            const double *hm = hs + mr * No;
            const double2 *gp = lds + c0 * P + pr;
            double2 v[kAhead];
            double h[2][kN3D];
            // element el = (l, n) of the walk over G^[l, c0 + n]
            auto read = [&](int el) {
                const int l = el / CB, n = el - l * CB;
                if (n == 0)
#pragma unroll
                    for (int i = 0; i < kN3D; ++i)
                        h[l & 1][i] = hm[i * NN + l];
                // past the last column of a ragged block: a column whose result is dropped
                v[el % kAhead] = gp[(l * No + (No % CB == 0 || c0 + n < No ? n : 0)) * P];
            };
#pragma unroll
            for (int el = 0; el < kAhead; ++el)
                read(el);
#pragma unroll
            for (int el = 0; el < No * CB; ++el) {
                const int l = el / CB, n = el - l * CB;
                const double2 g = v[el % kAhead];
#pragma unroll
                for (int i = 0; i < kN3D; ++i) {
                    xr[i][n] = fma(h[l & 1][i], g.x, xr[i][n]);
                    xi[i][n] = fma(h[l & 1][i], g.y, xi[i][n]);
                    pin(xr[i][n]);
                    pin(xi[i][n]);
                }
                if (el + kAhead < No * CB)
                    read(el + kAhead);
                __builtin_amdgcn_sched_barrier(0);
            }
            if (cb == NC - 1) {
                __syncthreads();  // every wave is done with G^ and dH of neighbour b
                if (bn < p.NB)
                    issue(bn);
            }
            double w[2][No];
            auto read_h = [&](int step) {
                const int j = step / CB, n = step % CB;
                const int nn = No % CB == 0 || c0 + n < No ? c0 + n : 0;
#pragma unroll
                for (int q = 0; q < No; ++q)
                    w[step & 1][q] = ht[(j * No + nn) * No + q];
            };
            read_h(0);
#pragma unroll
            for (int step = 0; step < kN3D * CB; ++step) {
                const int j = step / CB, n = step % CB;
                double tr = 0.0, ti = 0.0;
#pragma unroll
                for (int i = 0; i < kN3D; ++i) {
                    tr = fma(d[i].x, xr[i][n], fma(-d[i].y, xi[i][n], tr));
                    ti = fma(d[i].x, xi[i][n], fma(d[i].y, xr[i][n], ti));
                }
                if (No % CB != 0 && c0 + n >= No)
                    tr = ti = 0.0;
                if (n == CB - 1 && j + 1 < kN3D)
#pragma unroll
                    for (int i = 0; i < kN3D; ++i)
                        d[i] = (db + ((size_t)i * kN3D + j + 1) * npt)[pr];
                __builtin_amdgcn_sched_barrier(0);
                __builtin_amdgcn_s_waitcnt(kWaitLgkm0);
                __builtin_amdgcn_sched_barrier(0);
                if (step + 1 < kN3D * CB)
                    read_h(step + 1);
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int q = 0; q < No; ++q) {
                    sr[q] = fma(tr, w[step & 1][q], sr[q]);
                    si[q] = fma(ti, w[step & 1][q], si[q]);
                }
            }
        }
        b = bn;
    }
    bool bad = false;
    if (act) {
        double2 *o = J.Sh() + (((size_t)blockIdx.y * J.s.nb + blk) * p.na_cap * NN + (size_t)al * NN + m * No) * npt +
                     pt0 + pt;
#pragma unroll
        for (int n = 0; n < No; ++n) {
            bad |= !(finite(sr[n]) && finite(si[n]));
            o[(size_t)n * npt] = make_double2(sr[n], si[n]);
        }
    }
    if (__any(bad) && (threadIdx.x & 63) == 0)
        atomicOr(J.flag(), kFlagAll);
}

__device__ __forceinline__ double mfma(double a, double b, double c)
{
    return __builtin_amdgcn_mfma_f64_4x4x4f64(a, b, c, 0, 0, 0);
}
// x of the lane that CTRL names within each four
template <int CTRL>
__device__ __forceinline__ double quad_perm(double x)
{
    const int2 v = __builtin_bit_cast(int2, x);
    return __builtin_bit_cast(double, make_int2(__builtin_amdgcn_mov_dpp(v.x, CTRL, 0xf, 0xf, true),
                                                __builtin_amdgcn_mov_dpp(v.y, CTRL, 0xf, 0xf, true)));
}
// the lower 32 lanes of x in both halves, and its upper 32
__device__ __forceinline__ void halves(double x, double *lower, double *upper)
{
    const uint2 v = __builtin_bit_cast(uint2, x);
    const auto a = __builtin_amdgcn_permlane32_swap(v.x, v.x, false, false);
    const auto b = __builtin_amdgcn_permlane32_swap(v.y, v.y, false, false);
    *lower = __builtin_bit_cast(double, make_uint2(a[0], b[0]));
    *upper = __builtin_bit_cast(double, make_uint2(a[1], b[1]));
}

// dH of nb neighbours as 4 x 4 tiles, zero past the last orbital; of a half tile also its
// rows and its columns of the directions 0 and 1 side by side.
template <int No>
__device__ __forceinline__ void stage_tiles(double *hs, const double *dH, int nb)
{
    constexpr int T = (No + 3) / 4, Tf = No / 4, F = speck::matrix_tiles(No);
    for (int i = threadIdx.x; i < nb * F * 16; i += kSB) {
        const int fb = i >> 4, b = fb / F, f = fb - b * F, l = i & 3, h = i >> 2 & 3;
        int d = f / (T * T), r = 4 * (f / T % T) + l, c = 4 * (f % T) + h;
        if (No % 4 == 2 && f >= kN3D * T * T) {
            const int e = f - kN3D * T * T;
            if (e < T) {
                d = l >> 1;
                r = 4 * Tf + (l & 1);
                c = 4 * e + h;
            } else {
                d = h >> 1;
                r = 4 * (e - T) + l;
                c = 4 * Tf + (h & 1);
            }
        }
        hs[i] = r < No && c < No ? dH[(b * kN3D + d) * No * No + r * No + c] : 0.0;
    }
}
// Element offsets of a lane's rows and columns of G^ in tile t (past the last: it again),
// and a tile column at a point (of a half one re or im alone).
template <int No, int T>
__device__ __forceinline__ void matrix_offsets(int npt, int lo, int hi, unsigned (&go)[T], unsigned (&co)[T])
{
#pragma unroll
    for (int t = 0; t < T; ++t) {
        go[t] = (unsigned)(min(4 * t + hi, No - 1) * No * npt);
        co[t] = (unsigned)(min(4 * t + (No % 4 == 2 && t == No / 4 ? lo & 1 : lo), No - 1) * npt);
    }
}
template <int No, int T>
__device__ __forceinline__ void matrix_read(const double2 *gb, unsigned pt, int col, int lo, const unsigned (&go)[T],
                                            const unsigned (&co)[T], double2 (&g)[T])
{
#pragma unroll
    for (int k = 0; k < T; ++k)
        if (No % 4 == 2 && col == No / 4)
            g[k].x = reinterpret_cast<const double *>(gb)[2 * (go[k] + co[col] + pt) + (lo >> 1)];
        else
            g[k] = gb[go[k] + co[col] + pt];
}

// The sandwich in the matrix form, v_mfma_f64_4x4x4: four products of 4 x 4 matrices, one
// per point, so that nothing is padded but the orbitals.  With M_i^T = G^T dH_i^T and
// S^T = sum_j dH_j T_j^T the instruction's result layout is that of its second operand:
// T_j, mixed from the M_i in the lanes that hold them, goes into the second product
// without leaving the registers, and dH in 4 x 4 tiles (LDS) serves both products.
// A wave has four points and all orbitals; per neighbour it reads G^ once, a tile
// column ahead, and D^ from LDS, where the workgroup's are staged with dH.
// Norb = 4 t + 2 would waste half of the last tile in each direction.  There the
// 2 columns take two directions i (first product) or re and im (second), the 2 rows of
// M re and im, and the contraction over them j = 0 and 1 at once: 240 of the 324
// matrix instructions at Norb 10 remain.
// Per four points and neighbour 240 matrix (16 cycles) and 290 vector fp64 instructions
// (4 cycles); they share the units (alone 75 and 61 TFLOP/s, interleaved no more).  One
// GPU's energy shard: 4.03 ms per component, the units busy 80 % at 2.2 GHz (row form:
// 4.53 ms); 97 atoms with 12 orbitals and six neighbours 0.56 ms, row form 0.79 ms.
// A third wave per SIMD spills (8.3 ms); dH held in registers 4.25 ms.
template <int No, typename A>
__global__ __launch_bounds__(kSB, No <= 8 ? 3 : 2) void k_spec_matrix(const A arg)
{
    extern __shared__ double2 lds[];
    const Job J = job(arg);
    const auto &p = *J.p;
    constexpr int NN = No * No, T = (No + 3) / 4;
    constexpr bool kHalf = No % 4 == 2;       // the last tile is a half one,
    constexpr int Tf = kHalf ? T - 1 : T;     // the first Tf are handled alike
    constexpr int F = speck::matrix_tiles(No);
    int al;
    int64_t x;
    if (!sandwich_place(J.bid, J.s.na, (int64_t)p.npg * J.s.nb, &al, &x))
        return;
    const int pg = (int)(x % p.npg), blk = (int)(x / p.npg);
    const int a = J.s.a0 + al, npt = p.npt, P = p.P;
    const int cap = min(p.NB, speck::matrix_neighbours(No));
    double *hs = reinterpret_cast<double *>(lds + cap * kNF * P);
    const int lane = threadIdx.x & 63, lo = lane & 3, hi = lane >> 4;
    const int pl = (threadIdx.x >> 6) * 4 + ((lane >> 2) & 3), p0 = pg * P;  // the lane's point, the first one
    const int rounds = min(P, npt - p0 + 15) >> 4;
    const double2 *Gh = J.Gh() + ((size_t)blockIdx.y * J.s.nb + blk) * p.NA * NN * npt;
    const double2 *Dh = J.Dh() + ((size_t)blockIdx.y * p.NA + a) * p.NB * kNF * npt;
    const_ptr<int32_t> neigh = ro(J.t.neigh) + (size_t)a * p.NB;
    unsigned go[T], co[T];
    matrix_offsets<No>(npt, lo, hi, go, co);
    auto next_valid = [&](int b, int end) {
        while (b < end && (unsigned)neigh[b] >= (unsigned)p.NA)
            ++b;
        return b;
    };
    auto rows = [&](int b) { return Gh + (size_t)neigh[b] * NN * npt; };
    double2 g[T];  // the next tile column of G^
    auto read_g = [&](const double2 *gb, unsigned pt, int mu) { matrix_read<No>(gb, pt, mu, lo, go, co, g); };
    double sr[T][T], si[T][T];
    bool bad = false;
    for (int b0 = 0; b0 < p.NB; b0 += cap) {
        const int b1 = min(p.NB, b0 + cap), first = next_valid(b0, b1);
        if (first < b1)
            read_g(rows(first), min(p0 + pl, npt - 1), 0);
        __syncthreads();
        for (int i = threadIdx.x; i < (b1 - b0) * kNF * P; i += kSB) {
            const int r = i / P;
            lds[i] = (Dh + ((size_t)b0 * kNF + r) * npt)[min(p0 + i - r * P, npt - 1)];
        }
        stage_tiles<No>(hs, J.t.dH + ((size_t)a * p.NB + b0) * kN3D * NN, b1 - b0);
        __syncthreads();
        for (int rd = 0; rd < rounds; ++rd) {
            if (b0 == 0)
#pragma unroll
                for (int u = 0; u < T; ++u)
#pragma unroll
                    for (int v = 0; v < T; ++v)
                        sr[u][v] = si[u][v] = 0.0;
            for (int b = first; b < b1;) {
                const int bn = next_valid(b + 1, b1);
                const double2 *gb = rows(b), *gn = rows(bn < b1 ? bn : first);
                const unsigned pt = min(p0 + rd * 16 + pl, npt - 1);
                const unsigned ptn = bn < b1 || rd + 1 == rounds ? pt : (unsigned)min(p0 + rd * 16 + 16 + pl, npt - 1);
                const double *hb = hs + (b - b0) * F * 16 + (hi * 4 + lo);
                const double2 *db = lds + (b - b0) * kNF * P + rd * 16 + pl;
                auto h = [&](int i, int u, int v) { return hb[((i * T + u) * T + v) * 16]; };
                auto hx = [&](int k) { return hb[(kN3D * T * T + k) * 16]; };
                auto kx = [&](int u) { return hb[(kN3D * T * T + T + u) * 16]; };
#pragma unroll
                for (int mu = 0; mu < T; ++mu) {
                    double2 c[T];
#pragma unroll
                    for (int k = 0; k < T; ++k)
                        c[k] = g[k];
                    if (mu + 1 < T)
                        read_g(gb, pt, mu + 1);
                    else
                        read_g(gn, ptn, 0);
                    double mr[kN3D][T], mi[kN3D][T];
                    const bool half = kHalf && mu == Tf;
#pragma unroll
                    for (int k = 0; k < T; ++k) {
                        auto both = [&](int i, int v, double w) {
                            mr[i][v] = mfma(c[k].x, w, k ? mr[i][v] : 0.0);
                            if (!half)
                                mi[i][v] = mfma(c[k].y, w, k ? mi[i][v] : 0.0);
                        };
#pragma unroll
                        for (int i = 0; i < kN3D; ++i)
#pragma unroll
                            for (int v = 0; v < Tf; ++v)
                                both(i, v, h(i, v, k));
                        if (kHalf) {
                            both(0, T - 1, hx(k));
                            both(2, T - 1, h(2, T - 1, k));
                        }
                    }
                    if (kHalf) {
                        mr[1][T - 1] = quad_perm<0xEE>(mr[0][T - 1]);
                        if (!half)
                            mi[1][T - 1] = quad_perm<0xEE>(mi[0][T - 1]);
                    }
                    if (half)
#pragma unroll
                        for (int i = 0; i < kN3D; ++i)
#pragma unroll
                            for (int v = 0; v < T; ++v)
                                halves(mr[i][v], &mr[i][v], &mi[i][v]);
#pragma unroll
                    for (int jj = 0; jj < (half ? 2 : kN3D); ++jj) {
                        // of a half tile the lanes' halves take j = 0 and 1, then all j = 2
                        double2 d[kN3D];
#pragma unroll
                        for (int i = 0; i < kN3D; ++i)
                            d[i] = db[(i * kN3D + (half ? jj ? 2 : lane >> 5 : jj)) * P];
                        auto w = [&](int u) { return half ? jj ? h(2, u, mu) : kx(u) : h(jj, u, mu); };
#pragma unroll
                        for (int v = 0; v < T; ++v) {
                            double tr = 0.0, ti = 0.0;
#pragma unroll
                            for (int i = 0; i < kN3D; ++i) {
                                tr = fma(d[i].x, mr[i][v], fma(-d[i].y, mi[i][v], tr));
                                ti = fma(d[i].x, mi[i][v], fma(d[i].y, mr[i][v], ti));
                            }
                            if (kHalf && v == Tf) {
                                const double o = quad_perm<0x44>(ti);
                                tr = lo < 2 ? tr : o;
                            }
#pragma unroll
                            for (int u = 0; u < T; ++u) {
                                sr[u][v] = mfma(w(u), tr, sr[u][v]);
                                if (!(kHalf && v == Tf))
                                    si[u][v] = mfma(w(u), ti, si[u][v]);
                            }
                        }
                    }
                }
                b = bn;
            }
            const int pt = p0 + rd * 16 + pl;
            if (b1 < p.NB || pt >= npt)
                continue;
            double2 *o = J.Sh() + (((size_t)blockIdx.y * J.s.nb + blk) * p.na_cap * NN + (size_t)al * NN) * npt + pt;
#pragma unroll
            for (int u = 0; u < T; ++u)
#pragma unroll
                for (int v = 0; v < T; ++v) {
                    const int m = 4 * u + hi, n = 4 * v + (kHalf && v == Tf ? lo & 1 : lo);
                    if (m >= No || n >= No)
                        continue;
                    double2 *to = o + (unsigned)((n * No + m) * npt);
                    if (kHalf && v == Tf) {
                        bad |= !finite(sr[u][v]);
                        reinterpret_cast<double *>(to)[lo >> 1] = sr[u][v];
                    } else {
                        bad |= !(finite(sr[u][v]) && finite(si[u][v]));
                        *to = make_double2(sr[u][v], si[u][v]);
                    }
                }
        }
    }
    if (__any(bad) && (threadIdx.x & 63) == 0)
        atomicOr(J.flag(), kFlagAll);
}

// The phonon self-energy (Eqs. (4)-(5)): P_ij[q, w] = sum_k sum_e tr(dH_i^T X[k + q, e + s_w, a]
// dH_j Y[k, e, f]) is a correlation over (k, e), so with X^ the transform of the shifted
// component and Y^ that of the opposite one at the negated point,
//   P^_ij[point] = tr(dH_i^T X^ dH_j Y^) = sum_m sum_n U_i[n, m] W_j[m, n],
//   W_j = dH_j Y^,  U_i = dH_i^T X^,
// summed over the energy blocks (block n: V energies of Y, and of X the L rows from
// e0 + smin).  As in k_spec_sandwich a workgroup takes P points of one atom and a lane
// one point and row m: W_j[m, :] comes from LDS, U_i[n, m] from the lane's column m of X^
// with wave-uniform dH_i, and the sum over m goes through LDS once per neighbour.
// The same pipelining, and the same bound: NA 256, NB 4, NE 270, Nkz 3, Norb 9, both
// components, 1.25 ms; vector units busy 74 % of the cycles, 85 % of their instructions
// FMAs.
template <int No, int CB, int W>
__global__ __launch_bounds__(kSB, W) void k_spec_pi(const SpecOne arg)
{
    extern __shared__ double2 lds[];
    const Job J = job(arg);
    const auto &p = *J.p;
    constexpr int kAhead = CB < 4 ? CB : 4;  // at most a row: h holds two
    constexpr int NN = No * No, P = kSB / No;
    constexpr int NC = (No + CB - 1) / CB;   // column blocks; the last may be ragged
    double *hs = reinterpret_cast<double *>(lds + (NN > kNF * No ? NN : kNF * No) * P);  // [3][No][No]
    int a;
    int64_t x;
    if (!sandwich_place(J.bid, p.NA, p.npg, &a, &x))
        return;
    const int pg = (int)x;
    const int pt0 = pg * P, npt = p.npt;
    const int tid = threadIdx.x, m = tid / P, pt = tid - m * P;
    const int np = min(P, npt - pt0);
    const bool act = m < No && pt < np;
    const int mr = act ? m : 0, pr = act ? pt : 0;
    const size_t comp = (size_t)blockIdx.y * J.s.nb * p.NA * NN * npt + pt0;
    double2 *Ph = J.Dh() + ((size_t)blockIdx.y * p.NA + a) * p.NB * kNF * npt + pt0;
    const_ptr<int32_t> neigh = ro(J.t.neigh) + (size_t)a * p.NB;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);

    // start the copies of neighbour b's Y^ points (those past the last point repeat it) and dH
    auto issue = [&](int blk, int b) {
        int t = tid;
        asm volatile("" : "+v"(t));  // recomputed per neighbour rather than held
        const char *g = reinterpret_cast<const char *>(J.Sh() + comp + ((size_t)blk * p.NA + neigh[b]) * NN * npt);
        uint32_t *dst = reinterpret_cast<uint32_t *>(lds) + wave * 64 * 4;
#pragma unroll
        for (int i = 0; i < (NN * P + kSB - 1) / kSB; ++i) {
            const int u = t + i * kSB, c = u / P, q = min(u - c * P, np - 1);
            if (NN * P % kSB == 0 || u < NN * P)
                lds_copy<4>(g + (unsigned)((c * npt + q) * 16), dst + i * kSB * 4);
        }
        const char *h = reinterpret_cast<const char *>(J.t.dH + ((size_t)a * p.NB + b) * kN3D * NN);
        uint32_t *hd = reinterpret_cast<uint32_t *>(hs) + wave * 64;
#pragma unroll
        for (int i = 0; i < (kN3D * NN * 2 + kSB - 1) / kSB; ++i)
            if (t + i * kSB < kN3D * NN * 2)
                lds_copy<1>(h + (unsigned)((t + i * kSB) * 4), hd + i * kSB);
    };

    for (int blk = 0; blk < J.s.nb; ++blk) {
        const bool add = J.s.blk0 + blk > 0;  // the first block's sums overwrite
        double2 xc[No];                       // column m of X^
        {
            const double2 *xg = J.Gh() + comp + ((size_t)blk * p.NA + a) * NN * npt;
#pragma unroll
            for (int l = 0; l < No; ++l)
                xc[l] = (xg + (size_t)l * No * npt)[(unsigned)(mr * npt + pr)];
        }
        for (int b = 0; b < p.NB; ++b) {
            double2 *po = Ph + (size_t)b * kNF * npt;
            if ((unsigned)neigh[b] >= (unsigned)p.NA) {
                for (int i = tid; i < kNF * P; i += kSB)
                    if (i % P < np && !add)
                        po[(size_t)(i / P) * npt + i % P] = make_double2(0.0, 0.0);
                continue;
            }
            __syncthreads();  // the previous neighbour's sums are read
            issue(blk, b);
            __syncthreads();
            const_ptr<double> ht = ro(J.dht() + ((size_t)a * p.NB + b) * kN3D * NN);
            double sr[kNF], si[kNF];
#pragma unroll
            for (int i = 0; i < kNF; ++i)
                sr[i] = si[i] = 0.0;
#pragma unroll 1
            for (int cb = 0; cb < NC; ++cb) {
                const int c0 = cb * CB;
                double xr[kN3D][CB], xi[kN3D][CB];  // W_j[m, c0 + n]
#pragma unroll
                for (int j = 0; j < kN3D; ++j)
#pragma unroll
                    for (int n = 0; n < CB; ++n)
                        xr[j][n] = xi[j][n] = 0.0;
                const double *hm = hs + mr * No;
                const double2 *gp = lds + c0 * P + pr;
                double2 v[kAhead];
                double h[2][kN3D];
                auto read = [&](int el) {
                    const int l = el / CB, n = el - l * CB;
                    if (n == 0)
#pragma unroll
                        for (int j = 0; j < kN3D; ++j)
                            h[l & 1][j] = hm[j * NN + l];
                    v[el % kAhead] = gp[(l * No + (No % CB == 0 || c0 + n < No ? n : 0)) * P];
                };
#pragma unroll
                for (int el = 0; el < kAhead; ++el)
                    read(el);
#pragma unroll
                for (int el = 0; el < No * CB; ++el) {
                    const int l = el / CB, n = el - l * CB;
                    const double2 g = v[el % kAhead];
#pragma unroll
                    for (int j = 0; j < kN3D; ++j) {
                        xr[j][n] = fma(h[l & 1][j], g.x, xr[j][n]);
                        xi[j][n] = fma(h[l & 1][j], g.y, xi[j][n]);
                        pin(xr[j][n]);
                        pin(xi[j][n]);
                    }
                    if (el + kAhead < No * CB)
                        read(el + kAhead);
                    __builtin_amdgcn_sched_barrier(0);
                }
                // step (i, n): dH_i[:, n] is read during the step before
                double w[2][No];
                auto read_h = [&](int step) {
                    const int i = step / CB, n = step % CB;
                    const int nn = No % CB == 0 || c0 + n < No ? c0 + n : 0;
#pragma unroll
                    for (int q = 0; q < No; ++q)
                        w[step & 1][q] = ht[(i * No + nn) * No + q];
                };
                read_h(0);
#pragma unroll
                for (int step = 0; step < kN3D * CB; ++step) {
                    const int i = step / CB, n = step % CB;
                    __builtin_amdgcn_sched_barrier(0);
                    __builtin_amdgcn_s_waitcnt(kWaitLgkm0);
                    __builtin_amdgcn_sched_barrier(0);
                    if (step + 1 < kN3D * CB)
                        read_h(step + 1);
                    __builtin_amdgcn_sched_barrier(0);
                    double ur = 0.0, ui = 0.0;
#pragma unroll
                    for (int q = 0; q < No; ++q) {
                        ur = fma(w[step & 1][q], xc[q].x, ur);
                        ui = fma(w[step & 1][q], xc[q].y, ui);
                    }
                    if (No % CB != 0 && c0 + n >= No)
                        ur = ui = 0.0;
#pragma unroll
                    for (int j = 0; j < kN3D; ++j) {
                        double &zr = sr[i * kN3D + j], &zi = si[i * kN3D + j];
                        zr = fma(ur, xr[j][n], fma(-ui, xi[j][n], zr));
                        zi = fma(ur, xi[j][n], fma(ui, xr[j][n], zi));
                    }
                }
            }
            __syncthreads();  // every wave is done with Y^
            if (m < No)
#pragma unroll
                for (int i = 0; i < kNF; ++i)
                    lds[(i * No + m) * P + pt] = make_double2(sr[i], si[i]);
            __syncthreads();
            for (int i = tid; i < kNF * P; i += kSB) {
                const int ij = i / P, q = i - ij * P;
                if (q >= np)
                    continue;
                double2 *o = po + (size_t)ij * npt + q;
                double2 s = add ? *o : make_double2(0.0, 0.0);
                for (int r = 0; r < No; ++r) {
                    const double2 t = lds[(ij * No + r) * P + q];
                    s.x += t.x;
                    s.y += t.y;
                }
                *o = s;
            }
        }
    }
}

// The same in the matrix form (see k_spec_matrix): with A = dH_j, B = Y^ and A = X^T,
// B = dH_i the results W_j[m, n] and U_i[n, m] of one tile (m, n) lie in the same lanes, so
// the nine traces are lane-local products; per neighbour their sums over a point's 16 lanes
// are two more matrix products, with columns and rows of ones.  Of a half tile the rows m
// hold j = 0 and 1 (W) or re and im (U), the columns n re and im (W) or i = 0 and 1 (U);
// such sums are kept apart until the end: px by i (lanes' halves j = 0, 1), py by j
// (halves of each four i = 0, 1), pz both.  240 matrix and 256 vector fp64 instructions
// per four points and neighbour at Norb 10, and 40 matrix instructions for the sums.
// NA = 128, NE = 500, otherwise as the device-scale problem: 5.08 ms per call, row form
// 5.41 ms; the CPU-scale configuration 40 us, row form 49 us.
template <int No>
__global__ __launch_bounds__(kSB, 2) void k_spec_pi_matrix(const SpecOne arg)
{
    extern __shared__ double2 lds[];
    const Job J = job(arg);
    const auto &p = *J.p;
    constexpr int NN = No * No, T = (No + 3) / 4;
    constexpr bool kHalf = No % 4 == 2;
    constexpr int Tf = kHalf ? T - 1 : T, F = speck::matrix_tiles(No);
    double *hs = reinterpret_cast<double *>(lds);
    int a;
    int64_t x;
    if (!sandwich_place(J.bid, p.NA, p.npg, &a, &x))
        return;
    const int pg = (int)x;
    const int npt = p.npt, P = p.P;
    const int cap = min(p.NB, speck::pi_matrix_neighbours(No));
    const int lane = threadIdx.x & 63, lo = lane & 3, hi = lane >> 4;
    const int pl = (threadIdx.x >> 6) * 4 + ((lane >> 2) & 3), p0 = pg * P;
    const int rounds = min(P, npt - p0 + 15) >> 4;
    const size_t comp = (size_t)blockIdx.y * J.s.nb * p.NA * NN * npt;
    double2 *Ph = J.Dh() + ((size_t)blockIdx.y * p.NA + a) * p.NB * kNF * npt;
    const_ptr<int32_t> neigh = ro(J.t.neigh) + (size_t)a * p.NB;
    unsigned go[T], co[T];
    matrix_offsets<No>(npt, lo, hi, go, co);
    auto read = [&](const double2 *gb, unsigned pt, int col, double2 (&g)[T]) {
        matrix_read<No>(gb, pt, col, lo, go, co, g);
    };
    const double e[kN3D] = {lo == 0 ? 1.0 : 0.0, lo == 1 ? 1.0 : 0.0, lo == 2 ? 1.0 : 0.0};
    const double e01 = hi < 2 ? e[0] : e[1];
    for (int blk = 0; blk < J.s.nb; ++blk) {
        const bool add = J.s.blk0 + blk > 0;  // the first block's sums overwrite
        const double2 *X = J.Gh() + comp + ((size_t)blk * p.NA + a) * NN * npt;
        const double2 *Y = J.Sh() + comp + (size_t)blk * p.NA * NN * npt;
        for (int b0 = 0; b0 < p.NB; b0 += cap) {
            const int b1 = min(p.NB, b0 + cap);
            if (blk == 0 || cap < p.NB) {
                __syncthreads();
                stage_tiles<No>(hs, J.t.dH + ((size_t)a * p.NB + b0) * kN3D * NN, b1 - b0);
                __syncthreads();
            }
            auto next_valid = [&](int b) {
                while (b < b1 && (unsigned)neigh[b] >= (unsigned)p.NA)
                    ++b;
                return b;
            };
            const int first = next_valid(b0);
            for (int rd = 0; rd < rounds; ++rd) {
                const int at = p0 + rd * 16 + pl;
                const unsigned pt = min(at, npt - 1);
                double2 x[T][T], g[T];
#pragma unroll
                for (int u = 0; u < T; ++u)
                    read(X, pt, u, x[u]);
                if (first < b1)
                    read(Y + (size_t)neigh[first] * NN * npt, pt, 0, g);
                for (int b = first; b < b1;) {
                    const int bn = next_valid(b + 1);
                    const double2 *yb = Y + (size_t)neigh[b] * NN * npt;
                    const double2 *yn = Y + (size_t)neigh[bn < b1 ? bn : b] * NN * npt;
                    const double *hb = hs + (b - b0) * F * 16, *hr = hb + hi * 4 + lo, *hc = hb + lo * 4 + hi;
                    double pr[kNF], pi[kNF], pxr[kN3D], pxi[kN3D], pyr[kN3D], pyi[kN3D], pzr = 0.0, pzi = 0.0;
#pragma unroll
                    for (int i = 0; i < kNF; ++i)
                        pr[i] = pi[i] = 0.0;
#pragma unroll
                    for (int i = 0; i < kN3D; ++i)
                        pxr[i] = pxi[i] = pyr[i] = pyi[i] = 0.0;
#pragma unroll
                    for (int v = 0; v < T; ++v) {
                        const bool hn = kHalf && v == Tf;
                        double2 y[T];
#pragma unroll
                        for (int k = 0; k < T; ++k)
                            y[k] = g[k];
                        if (v + 1 < T)
                            read(yb, pt, v + 1, g);
                        else
                            read(yn, pt, 0, g);
#pragma unroll
                        for (int u = 0; u < T; ++u) {
                            const bool hm = kHalf && u == Tf;
                            const int nj = hm ? 2 : kN3D, ni = hn ? 2 : kN3D;
                            double wr[kN3D], wi[kN3D], ur[kN3D], ui[kN3D];
#pragma unroll
                            for (int k = 0; k < T; ++k) {
#pragma unroll
                                for (int j = 0; j < nj; ++j) {
                                    const double h = hm && j == 0 ? hr[(kN3D * T * T + k) * 16]
                                                                  : hr[(((hm ? 2 : j) * T + u) * T + k) * 16];
                                    wr[j] = mfma(h, y[k].x, k ? wr[j] : 0.0);
                                    if (!hn)
                                        wi[j] = mfma(h, y[k].y, k ? wi[j] : 0.0);
                                }
#pragma unroll
                                for (int i = 0; i < ni; ++i) {
                                    const double h = hn && i == 0 ? hc[(kN3D * T * T + T + k) * 16]
                                                                  : hc[(((hn ? 2 : i) * T + k) * T + v) * 16];
                                    ur[i] = mfma(x[u][k].x, h, k ? ur[i] : 0.0);
                                    if (!hm)
                                        ui[i] = mfma(x[u][k].y, h, k ? ui[i] : 0.0);
                                }
                            }
#pragma unroll
                            for (int j = 0; j < nj; ++j)
                                if (hn) {
                                    wi[j] = quad_perm<0xEE>(wr[j]);
                                    wr[j] = quad_perm<0x44>(wr[j]);
                                }
#pragma unroll
                            for (int i = 0; i < ni; ++i)
                                if (hm)
                                    halves(ur[i], &ur[i], &ui[i]);
#pragma unroll
                            for (int i = 0; i < ni; ++i)
#pragma unroll
                                for (int j = 0; j < nj; ++j) {
                                    const bool si = hn && i == 0, sj = hm && j == 0;  // two at once
                                    const int ii = hn ? 2 : i, jj = hm ? 2 : j;
                                    double &zr = si && sj ? pzr : si ? pyr[jj] : sj ? pxr[ii] : pr[ii * kN3D + jj];
                                    double &zi = si && sj ? pzi : si ? pyi[jj] : sj ? pxi[ii] : pi[ii * kN3D + jj];
                                    zr = fma(ur[i], wr[j], fma(-ui[i], wi[j], zr));
                                    zi = fma(ur[i], wi[j], fma(ui[i], wr[j], zi));
                                }
                        }
                    }
                    // over the lanes' hi: column j of i's tile; then over their lo: row i
                    double2 s = make_double2(0.0, 0.0), q = s;
#pragma unroll
                    for (int i = 0; i < kN3D; ++i) {
                        double2 r = make_double2(0.0, 0.0);
#pragma unroll
                        for (int j = 0; j < kN3D; ++j) {
                            r.x = mfma(pr[i * kN3D + j], e[j], r.x);
                            r.y = mfma(pi[i * kN3D + j], e[j], r.y);
                        }
                        if (kHalf) {
                            r.x = mfma(pxr[i], e01, r.x);
                            r.y = mfma(pxi[i], e01, r.y);
                            q.x = mfma(pyr[i], e[i], q.x);
                            q.y = mfma(pyi[i], e[i], q.y);
                        }
                        s.x = mfma(e[i], r.x, s.x);
                        s.y = mfma(e[i], r.y, s.y);
                    }
                    if (kHalf) {
                        q.x = mfma(pzr, e01, q.x);
                        q.y = mfma(pzi, e01, q.y);
                        s.x = mfma(e01, q.x, s.x);
                        s.y = mfma(e01, q.y, s.y);
                    }
                    if (hi < kN3D && lo < kN3D && at < npt) {
                        double2 *o = Ph + ((size_t)b * kNF + hi * kN3D + lo) * npt + at;
                        const double2 old = add ? *o : make_double2(0.0, 0.0);
                        *o = make_double2(old.x + s.x, old.y + s.y);
                    }
                    b = bn;
                }
                if (!add)
                    for (int b = b0; b < b1; ++b)
                        if ((unsigned)neigh[b] >= (unsigned)p.NA && hi < kN3D && lo < kN3D && at < npt)
                            Ph[((size_t)b * kNF + hi * kN3D + lo) * npt + at] = make_double2(0.0, 0.0);
            }
        }
    }
}

// Pi[q, w, a, b, i, j] = beta / (Nkz L) sum_kappa sum_eps P^_ij[kappa, eps]
// exp(2 pi i (kappa q / Nkz + eps (s_w - smin) / L)), one workgroup per (a, b, i, j): the
// eps sum per (kappa, w), split over 2^lg neighbouring lanes where there are few of them,
// then the kappa sum per (q, w).  The guard (SpecGuard): the peak of an atom and neighbour is
// the rms of the correlation over all its lags, those of no (q, w) among them, which is the
// root of sum |P^|^2; the direct kernel compares its outputs with that.  Also the
// neighbour-table check.
__global__ __launch_bounds__(kSB) void k_spec_pi_out(const SpecOne arg)
{
    extern __shared__ double2 lds[];
    const Job J = job(arg);
    const auto &p = *J.p;
    const int L = p.L, Nkz = p.Nkz, Nw = p.Nw, tid = threadIdx.x;
    double2 *tw = lds;                // [L]
    double2 *twk = tw + L;            // [Nkz]
    double2 *ph = twk + Nkz;          // [Nkz][L + 1]
    double2 *A = ph + Nkz * (L + 1);  // [Nkz][Nw]
    const int64_t ab = J.bid / kNF;
    const int ij = (int)(J.bid - ab * kNF);
    const int a = (int)(ab / p.NB), b = (int)(ab - (int64_t)a * p.NB);
    if (blockIdx.y == 0 && ij == 0 && tid == 0) {
        const int f = J.t.neigh[ab];
        if (f < 0 || f >= p.NA)
            atomicOr(arg.status, kStatusBadNeigh);
    }
    fill_twiddles(tw, L, 1, L);
    fill_twiddles(twk, Nkz, 1, Nkz);
    const double2 *src = J.Dh() + (((size_t)blockIdx.y * p.NA * p.NB + ab) * kNF + ij) * p.npt;
    double sum = 0.0;
    for (int i = tid; i < p.npt; i += kSB) {
        const double2 v = src[i];
        ph[i + i / L] = v;
        sum = fma(v.x, v.x, fma(v.y, v.y, sum));
    }
    __shared__ double s_sum[kSB / 64];
    __shared__ uint32_t s_top;
    auto spread = [&](double x) {
        for (int m = 1; m < 64; m <<= 1)
            x += __shfl_xor(x, m);
        if ((tid & 63) == 0)
            s_sum[tid >> 6] = x;
    };
    auto root = [&] {  // of the workgroup's sum, to 6 %: half the exponent
        double x = s_sum[0];
        for (int i = 1; i < kSB / 64; ++i)
            x += s_sum[i];
        return (magnitude(x) >> 1) + (1023u << 19);
    };
    spread(sum);
    __syncthreads();
    int lg = 0;
    while (lg < 4 && (Nkz * Nw << (lg + 1)) <= kSB)
        ++lg;
    const int G = 1 << lg, part = tid & (G - 1);
    // the lanes of a group take the same trips: the bound is a multiple of the group
    for (int i = tid >> lg; i < Nkz * Nw; i += kSB >> lg) {
        const int k = i / Nw, w = i - k * Nw, t0 = p.shift[w] - p.smin, st = (t0 << lg) % L;
        double xr = 0.0, xi = 0.0;
        int j = t0 * part % L;
        for (int e = part; e < L; e += G) {
            const double2 v = ph[k * (L + 1) + e], t = tw[j];  // t conjugated
            xr = fma(v.x, t.x, fma(v.y, t.y, xr));
            xi = fma(v.y, t.x, fma(-v.x, t.y, xi));
            j += st;
            j -= j >= L ? L : 0;
        }
        for (int h = 1; h < G; h <<= 1) {
            xr += __shfl_xor(xr, h);
            xi += __shfl_xor(xi, h);
        }
        if (part == 0)
            A[i] = make_double2(xr, xi);
    }
    __syncthreads();
    uint32_t peak = root();
    if (peak < (1023u - 450u) << 20 || peak > (1023u + 450u) << 20) {  // squares out of range: of values near one
        if (tid == 0)
            s_top = 0u;
        __syncthreads();
        uint32_t top = 0u;
        for (int i = tid; i < p.npt; i += kSB)
            top = max(top, magnitude(ph[i + i / L]));
        atomicMax(&s_top, top);
        __syncthreads();
        top = s_top;
        const int ex = (int)(top >> 20) - 1023;
        sum = 0.0;
        for (int i = tid; i < p.npt; i += kSB) {
            const double vr = ldexp(ph[i + i / L].x, -ex), vi = ldexp(ph[i + i / L].y, -ex);
            sum = fma(vr, vr, fma(vi, vi, sum));
        }
        spread(sum);
        __syncthreads();
        peak = top == 0u ? 0u : root() + (uint32_t)(ex << 20);
    }
    if (tid == 0)
        J.peaks()[(int64_t)(J.s.c0 + blockIdx.y) * p.NA * p.NB * kNF + J.bid] = peak;
    double2 *Pi = (double2 *)J.t.Sigma + (size_t)blockIdx.y * p.Nqz * Nw * p.NA * (p.NB + 1) * kNF;
    const double sc = 1.0 / ((double)Nkz * L), br = p.alpha_re * sc, bi = p.alpha_im * sc;
    bool bad = false;
    for (int i = tid; i < p.Nqz * Nw; i += kSB) {
        const int q = i / Nw, w = i - q * Nw;
        double xr = 0.0, xi = 0.0;
        int j = 0;
        for (int k = 0; k < Nkz; ++k) {
            const double2 v = A[k * Nw + w], t = twk[j];  // t conjugated
            xr = fma(v.x, t.x, fma(v.y, t.y, xr));
            xi = fma(v.y, t.x, fma(-v.x, t.y, xi));
            j += q;
            j -= j >= Nkz ? Nkz : 0;
        }
        bad |= !(finite(xr) && finite(xi));
        Pi[(((size_t)q * Nw + w) * p.NA + a) * (p.NB + 1) * kNF + b * kNF + ij] =
            make_double2(br * xr - bi * xi, br * xi + bi * xr);
    }
    if (__any(bad) && (tid & 63) == 0)
        atomicOr(J.flag(), kFlagAll);
}

template <typename K>
hipError_t allow_lds(K kernel, size_t bytes, bool &done)
{
    if (done)
        return hipSuccess;
    const hipError_t e = hipFuncSetAttribute((const void *)kernel, hipFuncAttributeMaxDynamicSharedMemorySize,
                                             (int)bytes);
    done = e == hipSuccess;
    return e;
}

struct Shape {
    dim3 grid;
    unsigned threads;
    size_t lds;
};

template <typename K, typename A>
hipError_t launch(K kernel, const A &arg, const Shape &h, bool &done, hipStream_t s)
{
    const hipError_t e = allow_lds(kernel, speck::kLdsOne, done);
    if (e != hipSuccess)
        return e;
    hipLaunchKernelGGL(kernel, h.grid, dim3(h.threads), h.lds, s, arg);
    return hipGetLastError();
}

template <typename T>
hipError_t prepare_launch(int L, const SpecOne &o, const Shape &h, hipStream_t s)
{
    hipError_t e = hipErrorInvalidValue;
    with_length(L, [&](auto r1, auto r2) {
        static bool done = false;
        e = launch(k_spec_prepare<T, decltype(r1)::value, decltype(r2)::value, SpecOne>, o, h, done, s);
    });
    return e;
}

template <typename T>
hipError_t inverse_launch(int L, const SpecOne &o, const Shape &h, hipStream_t s)
{
    hipError_t e = hipErrorInvalidValue;
    with_length(L, [&](auto r1, auto r2) {
        static bool done = false;
        e = launch(k_spec_inverse<T, decltype(r1)::value, decltype(r2)::value, SpecOne>, o, h, done, s);
    });
    return e;
}

// Columns per block and waves per SIMD of the row form: half the columns keep M, S^ and D^
// of a lane within 168 registers up to 10 orbitals, so that three waves share a SIMD; above,
// two waves' 256 registers hold them.  NA 256, NB 4, NE 270, Nkz 3, us per component: Norb 6
// 214 (all columns at two waves 222), 9 626 (677), 13 1766 (three waves 3104), 16 2511
// (14545: registers spill); Pi, both components, Norb 9 1252 (1771), 13 3460 (6542).  At
// Norb 5 two waves are as fast as three (148 and 147).
constexpr int col_block(int No) { return No <= 5 ? No : (No + 1) / 2; }
constexpr int waves(int No) { return No <= 10 ? 3 : 2; }

template <int No, typename A>
hipError_t sandwich_launch(int norb, const A &arg, const Shape &h, hipStream_t s)
{
    if (norb == No) {
        static bool done = false;
        if constexpr (speck::matrix_form(No))
            return launch(k_spec_matrix<No, A>, arg, h, done, s);
        else
            return launch(k_spec_sandwich<No, col_block(No), waves(No), A>, arg, h, done, s);
    }
    if constexpr (No < speck::kMaxNorb)
        return sandwich_launch<No + 1>(norb, arg, h, s);
    return hipErrorInvalidValue;
}

size_t dhat_lds(const SpecParams &p) { return ((size_t)p.Nw * kNF + p.L + p.Nqz) * sizeof(double2); }
int64_t prepare_wgs(const SpecParams &p, int jobs, int nb)
{
    return (jobs & kDht ? dht_wgs(p) : 0) + (jobs & kDhat ? dhat_wgs(p) : 0) +
           (jobs & kTransform ? fft_wgs(p, p.NA, nb) : 0);
}
// Up to this many D^ workgroups go with the transforms (four to a compute unit).
constexpr int64_t kTogether = 1024;

template <typename T>
hipError_t sigma_passes(SpecOne o, const SpectralGeom &g, hipStream_t s)
{
    const SpecParams &p = o.p;
    o.s.e_off = -p.smax;
    o.s.nrow = p.L;
    o.s.src_c = p.g_elems;
    o.s.dst = p.off_g;
    (void)hipGetLastError();
    hipError_t e = hipSuccess;
    const char *G = (const char *)o.t.G, *D = (const char *)o.t.D;
    char *S = (char *)o.t.Sigma;
    const size_t plus = dhat_lds(p);
    for (int c = 0; c < p.ncomp && e == hipSuccess; c += g.nc) {
        const unsigned nc = (unsigned)std::min(g.nc, p.ncomp - c);
        o.t.G = G + (size_t)c * p.g_elems * sizeof(T);
        o.t.D = D + (size_t)c * p.d_elems * sizeof(T);
        o.t.Sigma = S + (size_t)c * p.g_elems * sizeof(T);
        o.s.c0 = c;
        o.jobs = kDhat | (c == 0 ? kDht : 0);
        if (dhat_wgs(p) * nc > kTogether) {
            e = prepare_launch<T>(g.L, o, Shape{dim3((unsigned)prepare_wgs(p, o.jobs, 0), nc), kSB, plus}, s);
            o.jobs = 0;
        }
        for (o.s.blk0 = 0; o.s.blk0 < g.nblk && e == hipSuccess; o.s.blk0 += g.nb) {
            o.s.nb = std::min(g.nb, g.nblk - o.s.blk0);
            o.jobs |= kTransform;
            const bool with = o.jobs & kDhat;
            Shape h{dim3((unsigned)prepare_wgs(p, o.jobs, o.s.nb), nc),
                    (unsigned)(with ? std::max(g.fft_threads, kSB) : g.fft_threads),
                    with ? std::max(g.fft_lds, plus) : g.fft_lds};
            e = prepare_launch<T>(g.L, o, h, s);
            o.jobs = 0;
            for (o.s.a0 = 0; o.s.a0 < p.NA && e == hipSuccess; o.s.a0 += g.na) {
                o.s.na = std::min(g.na, p.NA - o.s.a0);
                e = sandwich_launch<1>(p.Norb, o, Shape{dim3((unsigned)sandwich_wgs(p, o.s.na, o.s.nb), nc), kSB,
                                                        g.sand_lds}, s);
                if (e == hipSuccess)
                    e = inverse_launch<T>(g.L, o, Shape{dim3((unsigned)(inverse_groups(p, o.s.na) * o.s.nb), nc),
                                                        (unsigned)g.fft_threads, g.fft_lds}, s);
            }
        }
    }
    return e;
}

// Lays out count(i) workgroups of each instance (rounded up to the eight XCDs).
template <typename Count>
unsigned lay_out(SpecMany *m, Count count)
{
    m->start[0] = 0;
    for (int i = 0; i < m->n; ++i)
        m->start[i + 1] = m->start[i] + (int32_t)((count(i) + 7) / 8 * 8);
    return (unsigned)m->start[m->n];
}

template <typename T>
hipError_t sigma_batch(SpecMany m, const SpecParams *hp, const SpectralGeom *const *g, hipStream_t s)
{
    const unsigned nc = (unsigned)hp[0].ncomp;
    Shape h{dim3(0, nc), kSB, 0};
    size_t lds = 0;
    for (int i = 0; i < m.n; ++i) {
        h.threads = std::max(h.threads, (unsigned)g[i]->fft_threads);
        h.lds = std::max(h.lds, g[i]->fft_lds);
        lds = std::max(lds, dhat_lds(hp[i]));
    }
    static bool d0 = false, d1 = false;
    int64_t dhat = 0;
    for (int i = 0; i < m.n; ++i)
        dhat += dhat_wgs(hp[i]);
    auto prepare = [&](int jobs, unsigned threads, size_t bytes) {
        m.jobs = jobs;
        const unsigned x = lay_out(&m, [&](int i) { return prepare_wgs(hp[i], jobs, hp[i].nblk); });
        return launch(k_spec_prepare<T, 0, 0, SpecMany>, m, Shape{dim3(x, nc), threads, bytes}, d0, s);
    };
    (void)hipGetLastError();
    hipError_t e;
    if (dhat * nc > kTogether) {
        e = prepare(kDht | kDhat, kSB, lds);
        if (e == hipSuccess)
            e = prepare(kTransform, h.threads, h.lds);
    } else {
        e = prepare(kDht | kDhat | kTransform, h.threads, std::max(h.lds, lds));
    }
    if (e != hipSuccess)
        return e;
    h.grid.x = lay_out(&m, [&](int i) { return sandwich_wgs(hp[i], hp[i].NA, hp[i].nblk); });
    size_t sand = 0;
    for (int i = 0; i < m.n; ++i)
        sand = std::max(sand, g[i]->sand_lds);
    e = sandwich_launch<1>(hp[0].Norb, m, Shape{h.grid, kSB, sand}, s);
    if (e != hipSuccess)
        return e;
    h.grid.x = lay_out(&m, [&](int i) { return inverse_groups(hp[i], hp[i].NA) * hp[i].nblk; });
    return launch(k_spec_inverse<T, 0, 0, SpecMany>, m, h, d1, s);
}

}  // namespace

hipError_t spectral_sigma_launch(const sse_desc &d, const SpectralGeom &g, const int32_t *w_shift,
                                 const sse_args &a, uint32_t *status, bool clear, uint32_t *host,
                                 const Fp64Params &redo, size_t redo_lds, void *ws, hipStream_t s)
{
    SpecOne o{};
    o.p = spectral_params(d, g, w_shift);
    o.t = SpecPtrs{a.neigh, a.dH, a.G, a.Dt, a.Sigma, (char *)ws};
    o.status = status;
    o.clear = clear;
    const bool c64 = d.prec != SSE_FP64;
    hipError_t e = c64 ? sigma_passes<float2>(o, g, s) : sigma_passes<double2>(o, g, s);
    if (e != hipSuccess)
        return e;
    Fp64Params r = redo;
    r.neigh = a.neigh;
    r.dH = a.dH;
    r.G = a.G;
    r.D = a.Dt;
    r.Sigma = a.Sigma;
    return fp64_redo_launch(r, c64, d.dt_antiherm != 0, redo_lds, d.ncomp, ws, status, host, s);
}

hipError_t spectral_batch_launch(int n, const sse_desc *const *d, const SpectralGeom *const *g,
                                 const sse_args *const *a, const size_t *ws_off, const SpecParams *hp,
                                 const SpecParams *params, const Fp64Params *redo, size_t redo_lds,
                                 uint32_t *status, bool clear, char *ws, hipStream_t s)
{
    if (n < 1 || n > kMaxBatch)
        return hipErrorInvalidValue;
    SpecMany m{};
    m.params = params;
    m.status = status;
    m.clear = clear;
    m.n = n;
    BatchLaunch bl{};
    bl.params = redo;
    bl.n = n;
    for (int i = 0; i < n; ++i) {
        m.t[i] = SpecPtrs{a[i]->neigh, a[i]->dH, a[i]->G, a[i]->Dt, a[i]->Sigma, ws + ws_off[i]};
        bl.ptr[i] = TensorPtrs{a[i]->neigh, a[i]->dH, a[i]->G, a[i]->Dt, a[i]->Sigma, m.t[i].ws};
    }
    const bool c64 = d[0]->prec != SSE_FP64;
    hipError_t e = c64 ? sigma_batch<float2>(m, hp, g, s) : sigma_batch<double2>(m, hp, g, s);
    return e != hipSuccess ? e : fp64_redo_batch_launch(bl, c64, d[0]->dt_antiherm != 0, redo_lds, d[0]->ncomp, s);
}

namespace {

constexpr int pi_col_block(int No) { return No <= 5 ? No : (No + 1) / 2; }
constexpr int pi_waves(int No) { return No <= 10 ? 3 : 2; }

template <int No>
hipError_t pi_sandwich_launch(const SpecOne &o, const Shape &h, hipStream_t s)
{
    if (o.p.Norb == No) {
        static bool done = false;
        if constexpr (speck::matrix_form(No))
            return launch(k_spec_pi_matrix<No>, o, h, done, s);
        else
            return launch(k_spec_pi<No, pi_col_block(No), pi_waves(No)>, o, h, done, s);
    }
    if constexpr (No < speck::kMaxNorb)
        return pi_sandwich_launch<No + 1>(o, h, s);
    return hipErrorInvalidValue;
}

}  // namespace

hipError_t spectral_pi_launch(const sse_desc &d, const SpectralGeom &g, const int32_t *w_shift,
                              const int32_t *neigh, const double *dH, const void *G, void *Pi, uint32_t *status,
                              void *ws, hipStream_t s)
{
    SpecOne o{};
    o.p = spectral_params(d, g, w_shift);
    o.t = SpecPtrs{neigh, dH, nullptr, nullptr, nullptr, (char *)ws};
    o.status = status;
    o.jobs = kDht;
    o.clear = 1;
    const SpecParams &p = o.p;
    const size_t pi_elems = (size_t)d.Nqz * d.Nw * d.NA * (d.NB + 1) * kNF;
    const size_t out_lds = ((size_t)g.L + d.Nkz + (size_t)d.Nkz * (g.L + 1) + (size_t)d.Nkz * d.Nw) * sizeof(double2);
    (void)hipGetLastError();
    hipError_t e = hipSuccess;
    const double2 *Gc = (const double2 *)G;
    for (int c = 0; c < d.ncomp && e == hipSuccess; c += g.nc) {
        const unsigned nc = (unsigned)std::min(g.nc, d.ncomp - c);
        o.s.c0 = c;
        o.t.G = Gc + (size_t)c * p.g_elems;
        o.t.D = Gc + (size_t)(1 - c) * p.g_elems;
        for (o.s.blk0 = 0; o.s.blk0 < g.nblk && e == hipSuccess; o.s.blk0 += g.nb) {
            o.s.nb = std::min(g.nb, g.nblk - o.s.blk0);
            const int64_t n = (o.jobs & kDht ? dht_wgs(p) : 0) + 2 * fft_wgs(p, p.NA, o.s.nb);
            const Shape h{dim3((unsigned)n, nc), (unsigned)g.fft_threads, g.fft_lds};
            e = hipErrorInvalidValue;
            with_length(g.L, [&](auto r1, auto r2) {
                static bool done = false;
                e = launch(k_spec_pi_prepare<decltype(r1)::value, decltype(r2)::value>, o, h, done, s);
            });
            if (e == hipSuccess)
                e = pi_sandwich_launch<1>(o, Shape{dim3((unsigned)sandwich_wgs(p, p.NA, 1), nc), kSB, g.sand_lds}, s);
            o.jobs = 0;
        }
        if (e != hipSuccess)
            break;
        o.t.Sigma = (double2 *)Pi + (size_t)c * pi_elems;
        static bool done = false;
        e = launch(k_spec_pi_out, o, Shape{dim3((unsigned)(d.NA * d.NB * kNF), nc), kSB, out_lds}, done, s);
    }
    return e;
}

}  // namespace sse
