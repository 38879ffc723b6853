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
//   k_spec_setup     status word, twiddle tables, dH transposed for scalar reads
//   k_spec_dhat      D^, and the neighbour-table check
//   k_spec_forward   G -> G^   (k and e transforms through LDS, one pass over memory)
//   k_spec_sandwich  G^, D^ -> S^
//   k_spec_inverse   S^ -> Sigma
// G^ and S^ are laid out [atom, orbital pair][kappa][eps], points fastest, so every
// pass reads and writes whole runs of points.  Rounding is that of binary64
// transforms: relative to the largest values of a block, as in any sum over them.
// Device scale (NA = 1024, NB = 4, Norb = 10, Nkz = Nqz = 7, NE = 1000, Nw = 30, both
// components, complex128): 1609 ms per call in the direct kernel, 84 ms here, of
// which the transforms (at the rate of a copy, 4.4 TB/s) 26 ms, the sandwich 57 ms.
// Inputs that are not finite, or so large that a transform overflows, raise a flag;
// the direct kernel then recomputes Sigma (its sums meet fewer elements).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstring>

#include "sse_copy.h"
#include "sse_dft.h"
#include "sse_spectral.h"

namespace sse {

namespace {

constexpr int kSB = speck::kSandBlock;
constexpr int kNkzReg = 8;  // momenta whose values a thread holds in registers

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

__device__ __forceinline__ bool finite(double x) { return __builtin_fabs(x) <= 1.7976931348623157e308; }

// A workgroup's instance, pass and index in it.
struct Job {
    const_ptr<SpecParams> p;
    SpecPtrs t;
    SpecPass s;
    int64_t bid, nwg;

    __device__ __forceinline__ uint32_t *flag() const { return reinterpret_cast<uint32_t *>(t.ws); }
    __device__ __forceinline__ double2 *tw() const { return reinterpret_cast<double2 *>(t.ws + p->off_tw); }
    __device__ __forceinline__ double *dht() const { return reinterpret_cast<double *>(t.ws + p->off_dht); }
    __device__ __forceinline__ double2 *Dh() const { return reinterpret_cast<double2 *>(t.ws + p->off_d); }
    __device__ __forceinline__ double2 *Gh() const { return reinterpret_cast<double2 *>(t.ws + p->off_g); }
    __device__ __forceinline__ double2 *Sh() const { return reinterpret_cast<double2 *>(t.ws + p->off_s); }
};
__device__ __forceinline__ Job job(const SpecOne &o)
{
    return Job{ro(&o.p), o.t, o.s, blockIdx.x, gridDim.x};
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
    const_ptr<SpecParams> p = ro(m.params) + m.idx[lo];
    return Job{p, m.t[lo], SpecPass{0, p->nblk, 0, p->NA, -p->smax, p->L, p->g_elems, p->off_g}, x - m.start[lo], m.start[lo + 1] - m.start[lo]};
}

// Flag and status word, twiddle tables and dH^T; a grid-stride loop over the latter.
template <typename A>
__global__ void k_spec_setup(const A arg)
{
    const Job J = job(arg);
    const auto &p = *J.p;
    const int64_t i0 = J.bid * blockDim.x + threadIdx.x;
    const int64_t step = J.nwg * blockDim.x;
    if (i0 == 0) {
        *J.flag() = 0u;
        if (arg.clear)
            *arg.status = 0u;
    }
    double2 *tw = J.tw();
    double *dht = J.dht();
    for (int64_t i = i0; i < p.L + p.Nkz * p.Nkz; i += step) {
        // the angle in (-1, 1] half turns
        const int n = i < p.L ? p.L : p.Nkz;
        int j = i < p.L ? (int)i : (int)(((i - p.L) / p.Nkz) * ((i - p.L) % p.Nkz) % p.Nkz);
        if (2 * j > n)
            j -= n;
        double s, c;
        sincospi(2.0 * j / n, &s, &c);
        tw[i] = make_double2(c, -s);
    }
    const int NN = p.NN, No = p.Norb;
    const int64_t nd = (int64_t)p.NA * p.NB * kN3D * NN;
    for (int64_t i = i0; i < nd; i += step) {
        const int64_t blk = i / NN;
        const int c = (int)(i - blk * NN), n = c / No, np = c - n * No;
        dht[i] = J.t.dH[blk * NN + np * No + n];
    }
}

// D^_ij[kappa, eps] of one (a, b) and kappa; the grid's y extent is the components.  The q sum goes
// into LDS (a few kB), then each thread takes an eps and all nine (i, j).
template <typename T, typename A>
__global__ __launch_bounds__(kSB) void k_spec_dhat(const A arg)
{
    extern __shared__ double2 lds[];
    const Job J = job(arg);
    const auto &p = *J.p;
    const int64_t ab = J.bid / p.Nkz;
    if (ab >= (int64_t)p.NA * p.NB)
        return;
    double2 *Dk = lds;                  // [Nw][9]
    double2 *tw = lds + p.Nw * kNF;     // [L]
    const int kap = (int)(J.bid - ab * p.Nkz), tid = threadIdx.x;
    const T *D = (const T *)J.t.D + (size_t)blockIdx.y * p.d_elems;
    const int64_t slab = (int64_t)p.NA * p.NB * kNF;
    if (kap == 0 && blockIdx.y == 0 && tid == 0) {
        const int f = J.t.neigh[ab];
        if (f < 0 || f >= p.NA)
            atomicOr(arg.status, kStatusBadNeigh);
    }
    for (int i = tid; i < p.L; i += kSB)
        tw[i] = J.tw()[i];
    const double2 *twk = J.tw() + p.L + kap * p.Nkz;
    for (int i = tid; i < p.Nw * kNF; i += kSB) {
        const int w = i / kNF, ij = i - w * kNF;
        // an anti-Hermitian D~ is completed from its entries i < j and Im of the diagonal
        const int ii = ij / kN3D, jj = ij - ii * kN3D;
        const bool low = p.antiherm && ii > jj, dia = p.antiherm && ii == jj;
        const T *src = D + ((int64_t)w * slab + ab * kNF + (low ? jj * kN3D + ii : ij));
        double xr = 0.0, xi = 0.0;
        for (int q = 0; q < p.Nqz; ++q) {
            double2 v = to_d2(src[(int64_t)q * p.Nw * slab]);
            if (low || dia)
                v.x = dia ? 0.0 : -v.x;
            const double2 t = twk[q];
            xr = fma(v.x, t.x, fma(-v.y, t.y, xr));
            xi = fma(v.x, t.y, fma(v.y, t.x, xi));
        }
        Dk[i] = make_double2(xr, xi);
    }
    __syncthreads();
    double2 *out = J.Dh() + ((size_t)blockIdx.y * p.NA * p.NB + ab) * kNF * p.npt + (size_t)kap * p.L;
    for (int e = tid; e < p.L; e += kSB) {
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

// The middle step of a transform of length R1 R2 in LDS: the R2-point transforms.
template <int R1, int R2, int S>
__device__ __forceinline__ void second_step(double2 *lds, int rows, int rowp)
{
    for (int it = threadIdx.x; it < rows * R1; it += blockDim.x) {
        const int row = it / R1, k1 = it - row * R1;
        double2 *x = lds + (size_t)row * rowp + k1 * (R2 + 1);
        double2 v[R2];
#pragma unroll
        for (int n = 0; n < R2; ++n)
            v[n] = x[n];
        dft::transform<R2, S>(v);
#pragma unroll
        for (int n = 0; n < R2; ++n)
            x[n] = v[n];
    }
}

// Sum over the Nkz rows of LDS at x (stride row) with the scalar factors w[k], conjugated if S > 0.
template <int S>
__device__ __forceinline__ double2 k_sum(const double2 (&v)[kNkzReg], const_ptr<double2> w, int Nkz)
{
    double xr = 0.0, xi = 0.0;
#pragma unroll
    for (int k = 0; k < kNkzReg; ++k)
        if (k < Nkz) {
            const double c = w[k].x, s = -S * w[k].y;
            xr = fma(v[k].x, c, fma(-v[k].y, s, xr));
            xi = fma(v[k].x, s, fma(v[k].y, c, xi));
        }
    return make_double2(xr, xi);
}

// Transform size L = R1 R2 as n = R2 n1 + n2, eps = k1 + R1 k2: R1-point transforms
// straight from global memory (R1 loads in flight per thread), twiddles, R2-point
// transforms in LDS, then the transform over k on the way out.  A workgroup takes C
// consecutive channels (64-byte pieces of each energy row) and all Nkz momenta.
// S is the sign of the exponents: -1, or +1 for the opposite component of the phonon
// self-energy, whose transform is wanted at the negated point.
template <typename T, int R1, int R2, int S, typename A>
__global__ __launch_bounds__(speck::kFftBlock, 4) void k_spec_forward(const A arg)
{
    extern __shared__ double2 lds[];
    constexpr int L = R1 * R2;
    const Job J = job(arg);
    const auto &p = *J.p;
    const int C = p.C, NC = p.NA * p.NN, Nkz = p.Nkz, rowp = p.rowp;
    const int ngrp = (NC + C - 1) >> p.logC;
    if (J.bid >= (int64_t)ngrp * J.s.nb)
        return;
    const int64_t x = xcd_remap(J.bid, (int64_t)ngrp * J.s.nb);
    const int blk = (int)(x / ngrp), ch0 = (int)(x - (int64_t)blk * ngrp) << p.logC;
    const T *src = (const T *)J.t.G + (int64_t)blockIdx.y * J.s.src_c;
    const double2 *tw = J.tw();
    const int ebase = (J.s.blk0 + blk) * p.V + J.s.e_off, nrow = J.s.nrow;
    for (int it = threadIdx.x; it < Nkz * C * R2; it += blockDim.x) {
        const int ch = it & (C - 1), r = it >> p.logC, k = r / R2, n2 = r - k * R2;
        const bool ok = ch0 + ch < NC;
        const T *row = src + (int64_t)k * p.NE * NC + ch0 + ch;
        double2 v[R1];
#pragma unroll
        for (int n1 = 0; n1 < R1; ++n1) {
            const int r = n1 * R2 + n2, e = ebase + r;
            v[n1] = ok && r < nrow && e >= 0 && e < p.NE ? to_d2(row[(int64_t)e * NC]) : make_double2(0.0, 0.0);
        }
        dft::transform<R1, S>(v);
        double2 *o = lds + (size_t)(k * C + ch) * rowp + n2;
        o[0] = v[0];
#pragma unroll
        for (int k1 = 1; k1 < R1; ++k1) {
            const double2 t = tw[k1 * n2];
            o[k1 * (R2 + 1)] = dft::cmul(v[k1], t.x, -S * t.y);
        }
    }
    __syncthreads();
    second_step<R1, R2, S>(lds, Nkz * C, rowp);
    __syncthreads();
    const_ptr<double2> twk = ro(tw + L);
    double2 *out = reinterpret_cast<double2 *>(J.t.ws + J.s.dst) + (((size_t)blockIdx.y * J.s.nb + blk) * NC + ch0) * p.npt;
    for (int it = threadIdx.x; it < L * C; it += blockDim.x) {
        const int ch = it / L, eps = it - ch * L;
        if (ch0 + ch >= NC)
            break;
        const double2 *y = lds + (size_t)ch * rowp + (eps % R1) * (R2 + 1) + eps / R1;
        double2 *o = out + (size_t)ch * p.npt + eps;
        if (Nkz <= kNkzReg) {
            double2 v[kNkzReg];
#pragma unroll
            for (int k = 0; k < kNkzReg; ++k)
                v[k] = k < Nkz ? y[(size_t)k * C * rowp] : make_double2(0.0, 0.0);
            for (int kap = 0; kap < Nkz; ++kap)
                o[(size_t)kap * L] = k_sum<S>(v, twk + kap * Nkz, Nkz);
        } else {
            for (int kap = 0; kap < Nkz; ++kap) {
                double xr = 0.0, xi = 0.0;
                for (int k = 0; k < Nkz; ++k) {
                    const double2 v = y[(size_t)k * C * rowp];
                    const double c = twk[kap * Nkz + k].x, s = -S * twk[kap * Nkz + k].y;
                    xr = fma(v.x, c, fma(-v.y, s, xr));
                    xi = fma(v.x, s, fma(v.y, c, xi));
                }
                o[(size_t)kap * L] = make_double2(xr, xi);
            }
        }
    }
}

// The same backwards: energies from points, then k on the way out, alpha and 1 / (Nkz L).
// An energy that no shift reaches gets an exact zero, as the direct sum gives.
template <typename T, int R1, int R2, typename A>
__global__ __launch_bounds__(speck::kFftBlock, 4) void k_spec_inverse(const A arg)
{
    extern __shared__ double2 lds[];
    constexpr int L = R1 * R2;
    const Job J = job(arg);
    const auto &p = *J.p;
    const int C = p.C, NC = J.s.na * p.NN, Nkz = p.Nkz, rowp = p.rowp;
    const int64_t strideE = (int64_t)p.NA * p.NN;
    const int ngrp = (NC + C - 1) >> p.logC;
    if (J.bid >= (int64_t)ngrp * J.s.nb)
        return;
    const int64_t x = xcd_remap(J.bid, (int64_t)ngrp * J.s.nb);
    const int blk = (int)(x / ngrp), ch0 = (int)(x - (int64_t)blk * ngrp) << p.logC;
    const double2 *tw = J.tw();
    const double2 *src = J.Sh() + (((size_t)blockIdx.y * J.s.nb + blk) * p.na_cap * p.NN + ch0) * p.npt;
    for (int it = threadIdx.x; it < Nkz * C * R2; it += blockDim.x) {
        const int row = it / R2, n2 = it - row * R2, ch = row & (C - 1), kap = row >> p.logC;
        const bool ok = ch0 + ch < NC;
        const double2 *y = src + (size_t)ch * p.npt + kap * L + n2;
        double2 v[R1];
#pragma unroll
        for (int n1 = 0; n1 < R1; ++n1)
            v[n1] = ok ? y[n1 * R2] : make_double2(0.0, 0.0);
        dft::transform<R1, 1>(v);
        double2 *o = lds + (size_t)row * rowp + n2;
        o[0] = v[0];
#pragma unroll
        for (int k1 = 1; k1 < R1; ++k1) {
            const double2 t = tw[k1 * n2];
            o[k1 * (R2 + 1)] = dft::cmul(v[k1], t.x, -t.y);
        }
    }
    __syncthreads();
    second_step<R1, R2, 1>(lds, Nkz * C, rowp);
    __syncthreads();
    const_ptr<double2> twk = ro(tw + L);
    const double sc = 1.0 / ((double)Nkz * L);
    const double ar = p.alpha_re * sc, ai = p.alpha_im * sc;
    const int e0 = (J.s.blk0 + blk) * p.V, nv = min(p.V, p.NE - e0);
    T *dst = (T *)J.t.Sigma + (size_t)blockIdx.y * p.g_elems + (size_t)J.s.a0 * p.NN + ch0;
    bool bad = false;
    for (int it = threadIdx.x; it < nv * C; it += blockDim.x) {
        const int ch = it & (C - 1), vv = it >> p.logC, e = e0 + vv;
        if (ch0 + ch >= NC)
            continue;
        bool reached = false;
        for (int w = 0; w < p.Nw && !reached; ++w)
            reached = e - p.shift[w] >= 0 && e - p.shift[w] < p.NE;
        const double2 *y = lds + (size_t)ch * rowp + (vv % R1) * (R2 + 1) + vv / R1;
        T *o = dst + (int64_t)e * strideE + ch;
        auto store = [&](int k, double2 s) {
            bad |= !(finite(s.x) && finite(s.y));
            if (reached)
                put(o + (int64_t)k * p.NE * strideE, ar * s.x - ai * s.y, ar * s.y + ai * s.x);
            else
                put(o + (int64_t)k * p.NE * strideE, 0.0, 0.0);
        };
        if (Nkz <= kNkzReg) {
            double2 v[kNkzReg];
#pragma unroll
            for (int kap = 0; kap < kNkzReg; ++kap)
                v[kap] = kap < Nkz ? y[(size_t)kap * C * rowp] : make_double2(0.0, 0.0);
            for (int k = 0; k < Nkz; ++k)
                store(k, k_sum<1>(v, twk + k * Nkz, Nkz));
        } else {
            for (int k = 0; k < Nkz; ++k) {
                double xr = 0.0, xi = 0.0;
                for (int kap = 0; kap < Nkz; ++kap) {
                    const double2 v = y[(size_t)kap * C * rowp];
                    const double c = twk[k * Nkz + kap].x, s = -twk[k * Nkz + kap].y;
                    xr = fma(v.x, c, fma(-v.y, s, xr));
                    xi = fma(v.x, s, fma(v.y, c, xi));
                }
                store(k, make_double2(xr, xi));
            }
        }
    }
    if (__any(bad) && (threadIdx.x & 63) == 0)
        atomicOr(J.flag(), 1u);
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
// Bound: binary64 FMA issue, and the power it takes.  At device scale (Norb = 10) the
// vector units are busy 72% of the cycles, 1560 of 1740 vector instructions per lane
// and neighbour are FMAs, LDS is busy 38% of the cycles, and the clock sinks from 2.4
// to 1.9 GHz: 3.6 ms per energy block of 160, 7.0 ms before the hand pipelining (FMA
// issue at 2.4 GHz: 1.9 ms).  Leaving out the copies, the scalar loads or the LDS
// reads shortens it by 8 to 14% each: none of them alone is what it waits for.
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
    // all XCDs work on one group of points at a time (its G^ rows stay in the
    // last-level cache); an XCD takes neighbouring atoms
    const int na8 = (J.s.na + 7) >> 3, per = na8 * 8;
    int64_t x = J.bid;
    const int in = (int)(x % per);
    x /= per;
    const int al = (in & 7) * na8 + (in >> 3);
    if (al >= J.s.na || x >= (int64_t)p.npg * J.s.nb)
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
        atomicOr(J.flag(), 1u);
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
// The same pipelining, and the same bound.  NA = 128, NE = 500, otherwise as the device-
// scale problem, both components: 204.6 ms per call in the direct kernel, 5.6 ms here, of
// which this kernel 3.9 ms and the four transforms 1.8 ms (the CPU-scale configuration:
// 1270 and 63 us).
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
    const int na8 = (p.NA + 7) >> 3, per = na8 * 8;
    const int in = (int)(J.bid % per), pg = (int)(J.bid / per);
    const int a = (in & 7) * na8 + (in >> 3);
    if (a >= p.NA || pg >= p.npg)
        return;
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

// Pi[q, w, a, b, i, j] = beta / (Nkz L) sum_kappa sum_eps P^_ij[kappa, eps]
// exp(2 pi i (kappa q / Nkz + eps (s_w - smin) / L)), one workgroup per (a, b, i, j): the
// eps sum per (kappa, w), split over 2^lg neighbouring lanes where there are few of them,
// then the kappa sum per (q, w).  Also the neighbour-table check.
__global__ __launch_bounds__(kSB) void k_spec_pi_out(const SpecOne arg)
{
    extern __shared__ double2 lds[];
    const Job J = job(arg);
    const auto &p = *J.p;
    const int L = p.L, Nkz = p.Nkz, Nw = p.Nw, tid = threadIdx.x;
    double2 *tw = lds;                // [L]
    double2 *ph = tw + L;             // [Nkz][L + 1]
    double2 *A = ph + Nkz * (L + 1);  // [Nkz][Nw]
    const int64_t ab = J.bid / kNF;
    const int ij = (int)(J.bid - ab * kNF);
    const int a = (int)(ab / p.NB), b = (int)(ab - (int64_t)a * p.NB);
    if (blockIdx.y == 0 && ij == 0 && tid == 0) {
        const int f = J.t.neigh[ab];
        if (f < 0 || f >= p.NA)
            atomicOr(arg.status, kStatusBadNeigh);
    }
    for (int i = tid; i < L; i += kSB)
        tw[i] = J.tw()[i];
    const double2 *src = J.Dh() + (((size_t)blockIdx.y * p.NA * p.NB + ab) * kNF + ij) * p.npt;
    for (int i = tid; i < p.npt; i += kSB)
        ph[i + i / L] = src[i];
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
    const_ptr<double2> twk = ro(J.tw() + L);
    double2 *Pi = (double2 *)J.t.Sigma + (size_t)blockIdx.y * p.Nqz * Nw * p.NA * (p.NB + 1) * kNF;
    const double sc = 1.0 / ((double)Nkz * L), br = p.alpha_re * sc, bi = p.alpha_im * sc;
    bool bad = false;
    for (int i = tid; i < p.Nqz * Nw; i += kSB) {
        const int q = i / Nw, w = i - q * Nw;
        double xr = 0.0, xi = 0.0;
        for (int k = 0; k < Nkz; ++k) {
            const double2 v = A[k * Nw + w];
            const double c = twk[q * Nkz + k].x, s = -twk[q * Nkz + k].y;
            xr = fma(v.x, c, fma(-v.y, s, xr));
            xi = fma(v.x, s, fma(v.y, c, xi));
        }
        bad |= !(finite(xr) && finite(xi));
        Pi[(((size_t)q * Nw + w) * p.NA + a) * (p.NB + 1) * kNF + b * kNF + ij] =
            make_double2(br * xr - bi * xi, br * xi + bi * xr);
    }
    if (__any(bad) && (tid & 63) == 0)
        atomicOr(J.flag(), 1u);
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

// Directions of the transforms: G to points, points to Sigma, and G to negated points.
enum Direction { kForward, kInverse, kOpposite };

template <Direction D, typename T, int R1, int R2, typename A>
hipError_t transform_as(const A &arg, const Shape &h, hipStream_t s)
{
    static bool done = false;
    auto launch = [&](auto kernel) {
        const hipError_t e = allow_lds(kernel, speck::kLdsOne, done);
        if (e != hipSuccess)
            return e;
        hipLaunchKernelGGL(kernel, h.grid, dim3(h.threads), h.lds, s, arg);
        return hipGetLastError();
    };
    if constexpr (D == kInverse)
        return launch(k_spec_inverse<T, R1, R2, A>);
    else
        return launch(k_spec_forward<T, R1, R2, D == kForward ? -1 : 1, A>);
}

template <Direction D, typename T, typename A>
hipError_t transform_launch(int L, const A &arg, const Shape &h, hipStream_t s)
{
    switch (L) {
    case 16: return transform_as<D, T, 4, 4>(arg, h, s);
    case 24: return transform_as<D, T, 4, 6>(arg, h, s);
    case 32: return transform_as<D, T, 4, 8>(arg, h, s);
    case 48: return transform_as<D, T, 6, 8>(arg, h, s);
    case 64: return transform_as<D, T, 8, 8>(arg, h, s);
    case 72: return transform_as<D, T, 8, 9>(arg, h, s);
    case 80: return transform_as<D, T, 8, 10>(arg, h, s);
    case 96: return transform_as<D, T, 8, 12>(arg, h, s);
    case 120: return transform_as<D, T, 10, 12>(arg, h, s);
    case 144: return transform_as<D, T, 12, 12>(arg, h, s);
    case 160: return transform_as<D, T, 10, 16>(arg, h, s);
    case 192: return transform_as<D, T, 12, 16>(arg, h, s);
    case 256: return transform_as<D, T, 16, 16>(arg, h, s);
    }
    return hipErrorInvalidValue;
}

// Columns per block and waves per SIMD of the sandwich kernel: half the columns keep
// M, S^ and D^ of a lane within 168 registers up to 10 orbitals, so that three waves
// share a SIMD.  At device scale 3.6 ms per energy block against 4.2 with all ten
// columns at two waves (a Norb of 12: 1.01 ms per call at two waves, 1.07 at three).
constexpr int col_block(int No) { return No <= 5 ? No : (No + 1) / 2; }
constexpr int waves(int No) { return No <= 10 ? 3 : 2; }

template <int No, typename A>
hipError_t sandwich_launch(int norb, const A &arg, const Shape &h, hipStream_t s)
{
    if (norb == No) {
        static bool done = false;
        const hipError_t e = allow_lds(k_spec_sandwich<No, col_block(No), waves(No), A>, speck::kLdsOne, done);
        if (e != hipSuccess)
            return e;
        hipLaunchKernelGGL((k_spec_sandwich<No, col_block(No), waves(No), A>), h.grid, dim3(h.threads), h.lds, s, arg);
        return hipGetLastError();
    }
    if constexpr (No < speck::kMaxNorb)
        return sandwich_launch<No + 1>(norb, arg, h, s);
    return hipErrorInvalidValue;
}

// Workgroups of one instance in each pass.
int64_t setup_wgs(const SpecParams &p)
{
    const int64_t n = (int64_t)p.NA * p.NB * kN3D * p.NN + p.L + p.Nkz * p.Nkz;
    return std::min<int64_t>((n + 255) / 256, 1024);
}
int64_t dhat_wgs(const SpecParams &p) { return (int64_t)p.NA * p.NB * p.Nkz; }
int64_t fft_wgs(const SpecParams &p, int64_t atoms, int nb) { return ((atoms * p.NN + p.C - 1) >> p.logC) * nb; }
int64_t sandwich_wgs(const SpecParams &p, int na, int nb) { return (int64_t)((na + 7) / 8 * 8) * p.npg * nb; }
size_t dhat_lds(const SpecParams &p) { return ((size_t)p.Nw * kNF + p.L) * sizeof(double2); }

template <typename T>
hipError_t sigma_passes(SpecOne o, const SpectralGeom &g, hipStream_t s)
{
    const SpecParams &p = o.p;
    o.s.e_off = -p.smax;
    o.s.nrow = p.L;
    o.s.src_c = p.g_elems;
    o.s.dst = p.off_g;
    (void)hipGetLastError();
    hipLaunchKernelGGL(k_spec_setup<SpecOne>, dim3((unsigned)setup_wgs(p)), dim3(256), 0, s, o);
    hipError_t e = hipGetLastError();
    const char *G = (const char *)o.t.G, *D = (const char *)o.t.D;
    char *S = (char *)o.t.Sigma;
    for (int c = 0; c < p.ncomp && e == hipSuccess; c += g.nc) {
        const unsigned nc = (unsigned)std::min(g.nc, p.ncomp - c);
        o.t.G = G + (size_t)c * p.g_elems * sizeof(T);
        o.t.D = D + (size_t)c * p.d_elems * sizeof(T);
        o.t.Sigma = S + (size_t)c * p.g_elems * sizeof(T);
        hipLaunchKernelGGL((k_spec_dhat<T, SpecOne>), dim3((unsigned)dhat_wgs(p), nc), dim3(kSB), dhat_lds(p), s, o);
        e = hipGetLastError();
        for (o.s.blk0 = 0; o.s.blk0 < g.nblk && e == hipSuccess; o.s.blk0 += g.nb) {
            o.s.nb = std::min(g.nb, g.nblk - o.s.blk0);
            Shape h{dim3((unsigned)fft_wgs(p, p.NA, o.s.nb), nc), (unsigned)g.fft_threads, g.fft_lds};
            e = transform_launch<kForward, T>(g.L, o, h, s);
            for (o.s.a0 = 0; o.s.a0 < p.NA && e == hipSuccess; o.s.a0 += g.na) {
                o.s.na = std::min(g.na, p.NA - o.s.a0);
                e = sandwich_launch<1>(p.Norb, o, Shape{dim3((unsigned)sandwich_wgs(p, o.s.na, o.s.nb), nc), kSB,
                                                        g.sand_lds}, s);
                h.grid.x = (unsigned)fft_wgs(p, o.s.na, o.s.nb);
                if (e == hipSuccess)
                    e = transform_launch<kInverse, T>(g.L, o, h, s);
            }
        }
    }
    return e;
}

// A launch over the instances of m that want() takes, count() workgroups each (rounded
// up to the eight XCDs); *any is whether there were some.
template <typename Want, typename Count>
unsigned lay_out(SpecMany *m, const SpecMany &all, Want want, Count count)
{
    m->n = 0;
    m->start[0] = 0;
    for (int i = 0; i < all.n; ++i)
        if (want(i)) {
            m->idx[m->n] = (uint8_t)i;
            m->t[m->n] = all.t[i];
            m->start[m->n + 1] = m->start[m->n] + (int32_t)((count(i) + 7) / 8 * 8);
            ++m->n;
        }
    return (unsigned)m->start[m->n];
}

template <typename T>
hipError_t sigma_batch(const SpecMany &all, const SpecParams *hp, const SpectralGeom *const *g, hipStream_t s)
{
    const unsigned nc = (unsigned)hp[0].ncomp;
    auto every = [](int) { return true; };
    SpecMany m = all;
    (void)hipGetLastError();
    unsigned x = lay_out(&m, all, every, [&](int i) { return setup_wgs(hp[i]); });
    hipLaunchKernelGGL(k_spec_setup<SpecMany>, dim3(x), dim3(256), 0, s, m);
    size_t lds = 0;
    for (int i = 0; i < all.n; ++i)
        lds = std::max(lds, dhat_lds(hp[i]));
    x = lay_out(&m, all, every, [&](int i) { return dhat_wgs(hp[i]); });
    hipLaunchKernelGGL((k_spec_dhat<T, SpecMany>), dim3(x, nc), dim3(kSB), lds, s, m);
    hipError_t e = hipGetLastError();
    auto transforms = [&](bool fwd) {
        bool done[kMaxBatch] = {};
        for (int i = 0; i < all.n && e == hipSuccess; ++i) {
            if (done[i])
                continue;
            Shape h{dim3(0, nc), 0, 0};
            h.grid.x = lay_out(&m, all,
                               [&](int j) {
                                   if (g[j]->L != g[i]->L)
                                       return false;
                                   done[j] = true;
                                   h.threads = std::max(h.threads, (unsigned)g[j]->fft_threads);
                                   h.lds = std::max(h.lds, g[j]->fft_lds);
                                   return true;
                               },
                               [&](int j) { return fft_wgs(hp[j], hp[j].NA, hp[j].nblk); });
            e = fwd ? transform_launch<kForward, T>(g[i]->L, m, h, s) : transform_launch<kInverse, T>(g[i]->L, m, h, s);
        }
    };
    transforms(true);
    if (e != hipSuccess)
        return e;
    x = lay_out(&m, all, every, [&](int i) { return sandwich_wgs(hp[i], hp[i].NA, hp[i].nblk); });
    e = sandwich_launch<1>(hp[0].Norb, m, Shape{dim3(x, nc), kSB, g[0]->sand_lds}, s);
    transforms(false);
    return e;
}

}  // namespace

hipError_t spectral_sigma_launch(const sse_desc &d, const SpectralGeom &g, const int32_t *w_shift,
                                 const sse_args &a, uint32_t *status, bool clear, const Fp64Params &redo,
                                 size_t redo_lds, void *ws, hipStream_t s)
{
    SpecOne o{};
    o.p = spectral_params(d, g, w_shift);
    o.t = SpecPtrs{a.neigh, a.dH, a.G, a.Dt, a.Sigma, (char *)ws};
    o.status = status;
    o.clear = clear;
    const bool c64 = d.prec != SSE_FP64;
    const size_t eb = c64 ? 8 : 16;
    hipError_t e = c64 ? sigma_passes<float2>(o, g, s) : sigma_passes<double2>(o, g, s);
    for (int c = 0; c < d.ncomp && e == hipSuccess; ++c) {
        Fp64Params r = redo;
        r.neigh = a.neigh;
        r.dH = a.dH;
        r.G = (const char *)a.G + (size_t)c * o.p.g_elems * eb;
        r.D = (const char *)a.Dt + (size_t)c * o.p.d_elems * eb;
        r.Sigma = (char *)a.Sigma + (size_t)c * o.p.g_elems * eb;
        e = fp64_redo_launch(r, c64, d.dt_antiherm != 0, redo_lds, (const uint32_t *)ws, s);
    }
    return e;
}

hipError_t spectral_batch_launch(int n, const sse_desc *const *d, const SpectralGeom *const *g,
                                 const sse_args *const *a, const size_t *ws_off, const SpecParams *hp,
                                 const SpecParams *params, const Fp64Params *redo, size_t redo_lds,
                                 uint32_t *status, char *ws, hipStream_t s)
{
    if (n < 1 || n > kMaxBatch)
        return hipErrorInvalidValue;
    SpecMany m{};
    m.params = params;
    m.status = status;
    m.n = n;
    for (int i = 0; i < n; ++i)
        m.t[i] = SpecPtrs{a[i]->neigh, a[i]->dH, a[i]->G, a[i]->Dt, a[i]->Sigma, ws + ws_off[i]};
    const bool c64 = d[0]->prec != SSE_FP64;
    hipError_t e = c64 ? sigma_batch<float2>(m, hp, g, s) : sigma_batch<double2>(m, hp, g, s);
    if (e != hipSuccess)
        return e;
    BatchLaunch bl{};
    bl.params = redo;
    bl.n = n;
    const size_t eb = c64 ? 8 : 16;
    for (int c = 0; c < d[0]->ncomp && e == hipSuccess; ++c) {
        for (int i = 0; i < n; ++i)
            bl.ptr[i] = TensorPtrs{a[i]->neigh, a[i]->dH, (const char *)a[i]->G + (size_t)c * hp[i].g_elems * eb,
                                   (const char *)a[i]->Dt + (size_t)c * hp[i].d_elems * eb,
                                   (char *)a[i]->Sigma + (size_t)c * hp[i].g_elems * eb, m.t[i].ws};
        e = fp64_redo_batch_launch(bl, c64, d[0]->dt_antiherm != 0, redo_lds, s);
    }
    return e;
}

namespace {

constexpr int pi_col_block(int No) { return No <= 5 ? No : (No + 1) / 2; }
constexpr int pi_waves(int No) { return No <= 10 ? 3 : 2; }

template <int No>
hipError_t pi_sandwich_launch(const SpecOne &o, const Shape &h, hipStream_t s)
{
    if (o.p.Norb == No) {
        static bool done = false;
        const hipError_t e = allow_lds(k_spec_pi<No, pi_col_block(No), pi_waves(No)>, speck::kLdsOne, done);
        if (e != hipSuccess)
            return e;
        hipLaunchKernelGGL((k_spec_pi<No, pi_col_block(No), pi_waves(No)>), h.grid, dim3(h.threads), h.lds, s, o);
        return hipGetLastError();
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
    o.clear = 1;
    const SpecParams &p = o.p;
    const size_t pi_elems = (size_t)d.Nqz * d.Nw * d.NA * (d.NB + 1) * kNF;
    const size_t out_lds = ((size_t)g.L + (size_t)d.Nkz * (g.L + 1) + (size_t)d.Nkz * d.Nw) * sizeof(double2);
    static bool done = false;
    hipError_t e = allow_lds(k_spec_pi_out, speck::kLdsOne, done);
    if (e != hipSuccess)
        return e;
    (void)hipGetLastError();
    hipLaunchKernelGGL(k_spec_setup<SpecOne>, dim3((unsigned)setup_wgs(p)), dim3(256), 0, s, o);
    e = hipGetLastError();
    const double2 *Gc = (const double2 *)G;
    for (int c = 0; c < d.ncomp && e == hipSuccess; c += g.nc) {
        const unsigned nc = (unsigned)std::min(g.nc, d.ncomp - c);
        for (o.s.blk0 = 0; o.s.blk0 < g.nblk && e == hipSuccess; o.s.blk0 += g.nb) {
            o.s.nb = std::min(g.nb, g.nblk - o.s.blk0);
            const Shape h{dim3((unsigned)fft_wgs(p, p.NA, o.s.nb), nc), (unsigned)g.fft_threads, g.fft_lds};
            o.t.G = Gc + (size_t)c * p.g_elems;
            o.s.e_off = p.smin;
            o.s.nrow = p.L;
            o.s.src_c = p.g_elems;
            o.s.dst = p.off_g;
            e = transform_launch<kForward, double2>(g.L, o, h, s);
            if (e != hipSuccess)
                break;
            o.t.G = Gc + (size_t)(1 - c) * p.g_elems;
            o.s.e_off = 0;
            o.s.nrow = p.V;
            o.s.src_c = -p.g_elems;
            o.s.dst = p.off_s;
            e = transform_launch<kOpposite, double2>(g.L, o, h, s);
            if (e == hipSuccess)
                e = pi_sandwich_launch<1>(o, Shape{dim3((unsigned)sandwich_wgs(p, p.NA, 1), nc), kSB, g.sand_lds}, s);
        }
        if (e != hipSuccess)
            break;
        o.t.Sigma = (double2 *)Pi + (size_t)c * pi_elems;
        hipLaunchKernelGGL(k_spec_pi_out, dim3((unsigned)(d.NA * d.NB * kNF), nc), dim3(kSB), out_lds, s, o);
        e = hipGetLastError();
    }
    return e;
}

}  // namespace sse
