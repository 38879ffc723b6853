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
    return Job{p, m.t[lo], SpecPass{0, p->nblk, 0, p->NA}, x - m.start[lo], m.start[lo + 1] - m.start[lo]};
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
template <typename T, int R1, int R2, typename A>
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
    const T *src = (const T *)J.t.G + (size_t)blockIdx.y * p.g_elems;
    const double2 *tw = J.tw();
    const int ebase = (J.s.blk0 + blk) * p.V - p.smax;
    for (int it = threadIdx.x; it < Nkz * C * R2; it += blockDim.x) {
        const int ch = it & (C - 1), r = it >> p.logC, k = r / R2, n2 = r - k * R2;
        const bool ok = ch0 + ch < NC;
        const T *row = src + (int64_t)k * p.NE * NC + ch0 + ch;
        double2 v[R1];
#pragma unroll
        for (int n1 = 0; n1 < R1; ++n1) {
            const int e = ebase + n1 * R2 + n2;
            v[n1] = ok && e >= 0 && e < p.NE ? to_d2(row[(int64_t)e * NC]) : make_double2(0.0, 0.0);
        }
        dft::transform<R1, -1>(v);
        double2 *o = lds + (size_t)(k * C + ch) * rowp + n2;
        o[0] = v[0];
#pragma unroll
        for (int k1 = 1; k1 < R1; ++k1) {
            const double2 t = tw[k1 * n2];
            o[k1 * (R2 + 1)] = dft::cmul(v[k1], t.x, t.y);
        }
    }
    __syncthreads();
    second_step<R1, R2, -1>(lds, Nkz * C, rowp);
    __syncthreads();
    const_ptr<double2> twk = ro(tw + L);
    double2 *out = J.Gh() + (((size_t)blockIdx.y * J.s.nb + blk) * NC + ch0) * p.npt;
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
                o[(size_t)kap * L] = k_sum<-1>(v, twk + kap * Nkz, Nkz);
        } else {
            for (int kap = 0; kap < Nkz; ++kap) {
                double xr = 0.0, xi = 0.0;
                for (int k = 0; k < Nkz; ++k) {
                    const double2 v = y[(size_t)k * C * rowp];
                    const double c = twk[kap * Nkz + k].x, s = twk[kap * Nkz + k].y;
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

template <typename T, int R1, int R2, typename A>
hipError_t transform_as(const A &arg, const Shape &h, bool fwd, hipStream_t s)
{
    static bool df = false, di = false;
    hipError_t e = fwd ? allow_lds(k_spec_forward<T, R1, R2, A>, speck::kLdsOne, df)
                       : allow_lds(k_spec_inverse<T, R1, R2, A>, speck::kLdsOne, di);
    if (e != hipSuccess)
        return e;
    if (fwd)
        hipLaunchKernelGGL((k_spec_forward<T, R1, R2, A>), h.grid, dim3(h.threads), h.lds, s, arg);
    else
        hipLaunchKernelGGL((k_spec_inverse<T, R1, R2, A>), h.grid, dim3(h.threads), h.lds, s, arg);
    return hipGetLastError();
}

template <typename T, typename A>
hipError_t transform_launch(int L, const A &arg, const Shape &h, bool fwd, hipStream_t s)
{
    switch (L) {
    case 16: return transform_as<T, 4, 4>(arg, h, fwd, s);
    case 24: return transform_as<T, 4, 6>(arg, h, fwd, s);
    case 32: return transform_as<T, 4, 8>(arg, h, fwd, s);
    case 48: return transform_as<T, 6, 8>(arg, h, fwd, s);
    case 64: return transform_as<T, 8, 8>(arg, h, fwd, s);
    case 72: return transform_as<T, 8, 9>(arg, h, fwd, s);
    case 80: return transform_as<T, 8, 10>(arg, h, fwd, s);
    case 96: return transform_as<T, 8, 12>(arg, h, fwd, s);
    case 120: return transform_as<T, 10, 12>(arg, h, fwd, s);
    case 144: return transform_as<T, 12, 12>(arg, h, fwd, s);
    case 160: return transform_as<T, 10, 16>(arg, h, fwd, s);
    case 192: return transform_as<T, 12, 16>(arg, h, fwd, s);
    case 256: return transform_as<T, 16, 16>(arg, h, fwd, s);
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
            e = transform_launch<T>(g.L, o, h, true, s);
            for (o.s.a0 = 0; o.s.a0 < p.NA && e == hipSuccess; o.s.a0 += g.na) {
                o.s.na = std::min(g.na, p.NA - o.s.a0);
                e = sandwich_launch<1>(p.Norb, o, Shape{dim3((unsigned)sandwich_wgs(p, o.s.na, o.s.nb), nc), kSB,
                                                        g.sand_lds}, s);
                h.grid.x = (unsigned)fft_wgs(p, o.s.na, o.s.nb);
                if (e == hipSuccess)
                    e = transform_launch<T>(g.L, o, h, false, s);
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
            e = transform_launch<T>(g[i]->L, m, h, fwd, s);
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

}  // namespace sse
