"""The kernels' constant tables (csrc/tables.h, run on the host) against their
closed forms in 60-digit decimal arithmetic.  Bars: the number of roundings of a
factor's own formula times 2^-53, with powers and products of l factors good to
one rounding."""
from __future__ import annotations

import ctypes
import os
import subprocess
from decimal import Decimal, getcontext

import numpy as np
import pytest

from paper_2111_13072_amd import build as B

U = 2.0 ** -53
SRC = r"""
#include "tables.h"
extern "C" void tables(double d, double eps_r, int L, double *tab, float *tab32, int *chl,
                       double *chn, double *chg)
{
    fill_tables(TableDst{tab, tab32, chl, chn, chg, d, eps_r, L, (L + 1) * (L + 1) - 1}, 0, 1);
}
extern "C" long tables_size(int L) { return (long)tables_len(L); }
extern "C" long tables32_size(int L) { return (long)tables32_len(L); }
extern "C" long offset(int which, int L)
{
    return (long)(which == 0 ? nf4_offset(L) : which == 1 ? lg4_offset(L) : fq4_offset(L));
}
"""


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    d = tmp_path_factory.mktemp("tables")
    src, out = str(d / "t.hip"), str(d / "t.so")
    with open(src, "w") as f:
        f.write(SRC)
    subprocess.run([B.hipcc(), f"--offload-arch={B.ARCH}", "-O2", "-std=c++17", "-fPIC", "-shared",
                    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops", "-w",
                    "-I", os.path.dirname(B.SRC), "-o", out, src], check=True)
    so = ctypes.CDLL(out)
    so.tables_size.restype = so.tables32_size.restype = so.offset.restype = ctypes.c_long
    return so


def _rel(x, exact):
    return abs(float((Decimal(float(x)) - exact) / exact))


@pytest.mark.parametrize("d,eps_r", [(0.25, 4.0), (0.05, 1.0), (0.9, 1.0), (0.01, 80.0), (0.5, 2.5)])
def test_tables_are_rounded_closed_forms(lib, d, eps_r):
    getcontext().prec = 60
    L = 64
    C = (L + 1) ** 2 - 1
    tab, tab32 = np.zeros(lib.tables_size(L)), np.zeros(lib.tables32_size(L), dtype=np.float32)
    chl, chn, chg = np.zeros(C, dtype=np.int32), np.zeros(C), np.zeros(C)
    ptr = lambda a: ctypes.c_void_p(a.ctypes.data)  # noqa: E731
    lib.tables(ctypes.c_double(d), ctypes.c_double(eps_r), L, ptr(tab), ptr(tab32), ptr(chl),
               ptr(chn), ptr(chg))
    n = L + 1
    ftil, wl, drive, selfw, selfw1 = (tab[k * n:(k + 1) * n] for k in range(5))
    lg4 = tab[lib.offset(1, L):][:4 * n].reshape(n, 4)
    fq4 = tab[lib.offset(2, L):].reshape(-1, 4)
    a, eps, four_pi = Decimal(1.0 - d), Decimal(eps_r), 4 * Decimal(float(np.pi))
    assert ftil[0] == 0.0 and drive[0] == 0.0
    p0 = Decimal(1)                               # P_{l-1}(0), l odd
    for l in range(1, n):
        a2l1, al1 = a ** (2 * l + 1), a ** (l + 1)
        den = (l + 1) * (eps - 1) * a2l1 + l * eps + l + 1
        f = (l * (eps - 1) + (l + eps + l * eps) * a2l1) / den
        # every term of f is positive: at most 6 roundings above, 5 below, the quotient
        assert _rel(ftil[l], f) <= 12 * U, l
        assert _rel(selfw[l], f / four_pi) <= 14 * U
        assert _rel(selfw1[l], (l + 1) * f / four_pi) <= 15 * U
        assert _rel(wl[l], Decimal(1) / (2 * l + 1)) <= U
        if l % 2:
            c = p0 * (Decimal(1) + Decimal(l) / (l + 1)) / 2
            bp = (2 * l + 1) * eps * al1 / den
            w = c * bp * (four_pi / (2 * l + 1)).sqrt()
            # c: a product of (l - 1) / 2 rounded quotients
            assert _rel(drive[l], w) <= (l + 17) * U, l
            p0 = -p0 * Decimal(l) / (l + 1)
        else:
            assert drive[l] == 0.0
        cl = Decimal(1)
        for k in range(1, l + 1):
            cl *= Decimal(2 * k - 1) / k
        assert _rel(lg4[l, 0], cl) <= 2 * U and _rel(lg4[l, 3], (2 * l + 1) * cl) <= 3 * U
    i, ch = 0, 0
    for m in range(n):
        norm2 = (Decimal(2) if m else Decimal(1)) / four_pi
        for k in range(1, m + 1):
            norm2 *= Decimal(2 * k + 1) / (2 * k)
        for l in range(m, n):
            if l > m:
                norm2 *= Decimal(4 * l * l - 1) / (l * l - m * m)
            if l >= m + 2:
                gamma = Decimal((l - 1) ** 2 - m * m) / ((2 * l - 1) * (2 * l - 3))
                assert _rel(fq4[i, 0], gamma) <= 2 * U
            else:
                assert fq4[i, 0] == 0.0
            assert fq4[i, 1] == l + 0.5
            i += 1
            for _ in range(0 if l == 0 else 2 if m else 1):
                assert chl[ch] == l
                assert _rel(chn[ch], norm2.sqrt()) <= 3 * U
                assert _rel(chg[ch], norm2 / (2 * l + 1)) <= 3 * U
                ch += 1
    assert ch == C and not fq4[i, :].any()
