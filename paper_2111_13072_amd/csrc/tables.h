// Constant tables of the kernels: the per-l and per-(l, m) coefficients, filled on
// the device (no copies: an evaluation without a handle fills them on each call).
// Plain arithmetic that also runs on the host, where the tests check it.
#ifndef MRPSIM_TABLES_H
#define MRPSIM_TABLES_H

#include <hip/hip_runtime.h>

#include <cmath>
#include <cstddef>

namespace {

constexpr double kPi = 3.14159265358979323846;

// Layout of the FP64 table block: five per-l arrays (ftil, wl, drive_w, self_w,
// self_w1), then at 32-byte aligned offsets the near-field constants (nf4, lg4)
// and the rescaled recurrence (fq4) with its zero entry.  The first offset is that
// of nine arrays and two (l, m) triangles, and the FP32 block starts two float4 per
// l in: the sizes are part of what sim_footprint_bytes reports and of which
// evaluations the static buffer takes, and stay what they were.
__host__ __device__ inline size_t nf4_offset(int L)
{
    const size_t base = (size_t)9 * (L + 1) + 2 * (size_t)((L + 1) * (L + 2) / 2);
    return (base + 3) & ~size_t(3);
}
__host__ __device__ inline size_t lg4_offset(int L) { return nf4_offset(L) + 4 * (size_t)(L + 1); }
__host__ __device__ inline size_t fq4_offset(int L) { return lg4_offset(L) + 4 * (size_t)(L + 1); }
// one zero entry after the fq4 triangle: the moments kernel reads one ahead
inline size_t tables_len(int L) { return fq4_offset(L) + 4 * (size_t)((L + 1) * (L + 2) / 2 + 1); }

// FP32 tables of the field kernel, each at a 16-byte aligned offset: the
// far-field recurrence and the full near field's Legendre constants.
__host__ __device__ inline size_t fq4_32_offset(int L) { return 8 * (size_t)(L + 1); }
__host__ __device__ inline size_t lw4_32_offset(int L)
{
    return fq4_32_offset(L) + 4 * (size_t)((L + 1) * (L + 2) / 2);
}
inline size_t tables32_len(int L) { return lw4_32_offset(L) + 4 * (size_t)(L + 1); }

struct TableDst {
    double *tab;
    float *tab32;
    int *chl;
    double *chn, *chg;
    double d, eps_r;
    int L, C;
};

// A product of exact factors with its rounding errors carried along: the
// tables' factors are good to about one rounding at any degree.
struct ExactProduct {
    double hi, lo = 0.0;
    __host__ __device__ void mul(double a)
    {
#pragma clang fp contract(off)
        const double p = hi * a;
        lo = fma(lo, a, fma(hi, a, -p));
        hi = p;
    }
    __host__ __device__ double times(const ExactProduct &o) const
    {
#pragma clang fp contract(off)
        const double p = hi * o.hi;
        return fma(hi, o.lo, fma(lo, o.hi, fma(hi, o.hi, -p))) + p;
    }
    __host__ __device__ double over(const ExactProduct &d) const
    {
#pragma clang fp contract(off)
        const double q = hi / d.hi;
        return fma(q, lo / hi - d.lo / d.hi, fma(-q, d.hi, hi) / d.hi) + q;
    }
};

// The entries i0, i0 + stride, ... of every table.  f_l and b^P_l are the
// closed forms of App. A and Sec. 3 (R = 1, R_E = 1 - d); c_l, the Legendre
// coefficients of the electrode data 1/2 sgn(cos th), are taken as
// (P_{l-1}(0) - P_{l+1}(0)) / 2.  Every entry comes from products of its own,
// so the threads share nothing; no contraction, so that the tables of two
// kernels are the same bits.
__host__ __device__ inline void fill_tables(const TableDst &t, int i0, int stride)
{
#pragma clang fp contract(off)
    const int L = t.L, n = L + 1, tri_n = (L + 1) * (L + 2) / 2;
    double *ftil = t.tab, *wl = ftil + n, *drive = wl + n, *selfw = drive + n,
           *selfw1 = selfw + n;
    double *nf4 = t.tab + nf4_offset(L), *lg4 = t.tab + lg4_offset(L), *fq4 = t.tab + fq4_offset(L);
    float *fq32 = t.tab32 + fq4_32_offset(L), *lw32 = t.tab32 + lw4_32_offset(L);
    for (int l = i0; l <= L; l += stride) {
        const double eps = t.eps_r, dl = (double)l, a = 1.0 - t.d;
        ExactProduct odd{1.0}, fac{1.0}, power{1.0};   // (2l-1)!!, l!, a^l
        for (int k = 1; k <= l; ++k) {
            odd.mul(2.0 * k - 1.0);
            fac.mul((double)k);
            power.mul(a);
        }
        ExactProduct next = power;
        next.mul(a);
        const double al1 = next.hi + next.lo, a2l1 = power.times(next);   // a^(l+1), a^(2l+1)
        const double f = (dl * (eps - 1.0) + (dl + eps + dl * eps) * a2l1) /
                         ((dl + 1.0 + dl * eps) + (dl + 1.0) * (eps - 1.0) * a2l1);
        const double bP = (2.0 * dl + 1.0) * eps * al1 /
                          ((dl + 1.0) * (eps - 1.0) * a2l1 + dl * eps + dl + 1.0);
        double c = 0.0;
        if (l & 1) {
            double p0 = 1.0;   // P_{l-1}(0); P_{l+1}(0) = -l / (l+1) P_{l-1}(0)
            for (int k = 1; k < l - 1; k += 2) p0 = -(double)k / (k + 1.0) * p0;
            c = 0.5 * (p0 - -dl / (dl + 1.0) * p0);
        }
        ftil[l] = l == 0 ? 0.0 : f;
        wl[l] = 1.0 / (2.0 * dl + 1.0);
        drive[l] = c * bP * sqrt(4.0 * kPi / (2.0 * dl + 1.0));
        selfw[l] = l == 0 ? 0.0 : f / (4.0 * kPi);
        selfw1[l] = selfw[l] * (dl + 1.0);
        nf4[4 * l + 0] = (2.0 * dl + 1.0) / (dl + 1.0);
        nf4[4 * l + 1] = dl / (dl + 1.0);
        nf4[4 * l + 2] = 2.0 * dl + 1.0;
        nf4[4 * l + 3] = dl;
        // P_l = c_l Ph_l with c_0 = 1, c_l = c_{l-1} (2l-1)/l: the three-term
        // recurrence l P_l = (2l-1) u P_{l-1} - (l-1) P_{l-2} becomes
        // Ph_l = u Ph_{l-1} - gamma_l Ph_{l-2}, gamma_l = (l-1)^2 / ((2l-1)(2l-3));
        // P'_{l+1} = P'_{l-1} + (2l+1) c_l Ph_l
        const double cl = odd.over(fac);
        lg4[4 * l + 0] = cl;
        lg4[4 * l + 1] = dl * cl;
        lg4[4 * l + 2] = dl * dl / ((2.0 * dl + 1.0) * (2.0 * dl - 1.0));
        lg4[4 * l + 3] = (2.0 * dl + 1.0) * cl;
        lw32[4 * l + 0] = (float)(1.0 / (dl + 1.0));
        lw32[4 * l + 1] = 0.0f;
        lw32[4 * l + 2] = (float)(2.0 * dl + 1.0);
        lw32[4 * l + 3] = (float)(dl + 1.0);
    }
    // (l, m) in stream order: Q_l^m = N_lm Qh_l^m, with N_lm^2 = (2 - [m = 0]) /
    // (4 pi) prod_{k <= m} (2k+1)/(2k) prod_{m < k <= l} (4k^2-1)/(k^2-m^2) and
    // gamma_lm = ((l-1)^2 - m^2) / ((2l-1)(2l-3))
    for (int i = i0; i <= tri_n; i += stride) {
        int m = 0, j = i;
        while (m < L && j >= n - m) {
            j -= n - m;
            ++m;
        }
        const int l = m + j;
        double gamma = 0.0, half = 0.0;
        if (i < tri_n) {
            half = (double)l + 0.5;
            if (l >= m + 2)
                gamma = (double)((l - 1) * (l - 1) - m * m) / ((2.0 * l - 1.0) * (2.0 * l - 3.0));
            fq32[4 * i] = (float)gamma;
            fq32[4 * i + 1] = (float)half;
            fq32[4 * i + 2] = 0.0f;
            fq32[4 * i + 3] = 0.0f;
        }
        fq4[4 * i] = gamma;
        fq4[4 * i + 1] = half;
        fq4[4 * i + 2] = 0.0;
        fq4[4 * i + 3] = 0.0;
        // the channels of this (l, m): cos, and sin for m > 0
        if (i == tri_n || l == 0) continue;
        const int ch = m == 0 ? l - 1 : L + (m - 1) * (2 * L + 2 - m) + 2 * (l - m);
        if (ch >= t.C) continue;   // axisymmetric: m = 0 only
        ExactProduct num{m > 0 ? 2.0 : 1.0}, den{4.0 * kPi};
        for (int k = 1; k <= m; ++k) {
            num.mul(2.0 * k + 1.0);
            den.mul(2.0 * k);
        }
        for (int k = m + 1; k <= l; ++k) {
            num.mul((double)(4 * k * k - 1));
            den.mul((double)(k * k - m * m));
        }
        const double n2 = num.over(den);
        for (int q = 0; q < (m > 0 ? 2 : 1); ++q) {
            t.chl[ch + q] = l;
            t.chn[ch + q] = sqrt(n2);
            t.chg[ch + q] = n2 / (2.0 * l + 1.0);   // a raw sum of Qh to a coefficient
        }
    }
    if (i0 == 0 && t.C == 0) {
        t.chl[0] = 0;
        t.chn[0] = 0.0;
        t.chg[0] = 0.0;
    }
}

}  // namespace

#endif  // MRPSIM_TABLES_H
