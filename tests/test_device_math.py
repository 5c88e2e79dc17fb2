"""The FP64 arithmetic of the device code, compiled for the host from the same
source: the HIP qualifiers are defined away and the hardware's builtins stand
as their documented behaviour (seeds with a relative error of 2^-23, the
division fix-up, the class test, the median of three)."""
import ctypes as C
import os
import subprocess

import numpy as np
import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_1110_0740_amd", "csrc")

SHIM = r"""
#include <math.h>
#include <stdint.h>
#include <string.h>
#include <type_traits>
#define __device__
#define __host__
#define __forceinline__ inline
static inline double bits(double x, double e)
{
    // a seed: the value with a relative error of up to 2^-23
    uint64_t u;
    memcpy(&u, &x, 8);
    return x * (1.0 + ((double)((u * 0x9E3779B97F4A7C15ull) >> 40) / 8388608.0 - 1.0) * e);
}
static inline double seed_rcp(double x) { return x == 0.0 || isinf(x) || isnan(x) ? 1.0 / x : bits(1.0 / x, 0x1p-23); }
static inline double seed_rsq(double x)
{
    return !(x > 0.0) || isinf(x) ? 1.0 / sqrt(x) : bits(1.0 / sqrt(x), 0x1p-23);
}
static inline double fixup(double q, double d, double n)
{
    const double s = copysign(1.0, d) * copysign(1.0, n);
    if (isnan(d) || isnan(n) || (d == 0.0 && n == 0.0) || (isinf(d) && isinf(n))) return NAN;
    if (d == 0.0 || isinf(n)) return s * INFINITY;
    if (isinf(d) || n == 0.0) return s * 0.0;
    return copysign(q, s);
}
static inline bool is_class(double x, int m)
{
    // bits 5 and 6: -0 and +0, 9: +infinity
    return ((m & 0x20) && x == 0.0 && signbit(x)) || ((m & 0x40) && x == 0.0 && !signbit(x)) ||
           ((m & 0x200) && isinf(x) && x > 0.0);
}
static inline float med3(float a, float b, float c) { return fmaxf(fminf(a, b), fminf(fmaxf(a, b), c)); }
#define __builtin_amdgcn_rcp seed_rcp
#define __builtin_amdgcn_rsq seed_rsq
#define __builtin_amdgcn_rsqf(x) (1.0f / sqrtf(x))
#define __builtin_amdgcn_div_fixup fixup
#define __builtin_amdgcn_class is_class
#define __builtin_amdgcn_fmed3f med3
namespace ctu {
// the reference precision
typedef long double ld;
static inline ld rcp(ld x) { return 1 / x; }
static inline ld quot(ld a, ld b) { return a / b; }
static inline ld root(ld x) { return sqrtl(x); }
static inline ld rsq(ld x) { return 1 / sqrtl(x); }
}
#include "ctu_device.hpp"
extern "C" {
void t_rcp(int n, const double *a, double *r) { for (int i = 0; i < n; i++) r[i] = ctu::rcp(a[i]); }
void t_quot(int n, const double *a, const double *b, double *r) { for (int i = 0; i < n; i++) r[i] = ctu::quot(a[i], b[i]); }
void t_root(int n, const double *a, double *r) { for (int i = 0; i < n; i++) r[i] = ctu::root(a[i]); }
void t_rsq(int n, const double *a, double *r) { for (int i = 0; i < n; i++) r[i] = ctu::rsq(a[i]); }
void t_mc(int n, const double *a, const double *b, double *r) { for (int i = 0; i < n; i++) r[i] = ctu::lim_mc(a[i], b[i]); }
// HLLD fluxes of n pairs of states (9 values each) along x: as the library
// forms them in FP64, in the jump form, and the jump form in long double,
// rounded to FP64 with its remainder
void t_hlld(int n, const double *L, const double *R, double gam, double *F, double *J, double *hi, double *lo)
{
    for (int i = 0; i < n; i++) {
        double s;
        ctu::hlld<0, double>(L + 9 * i, R + 9 * i, F + 9 * i, s, gam, 1.0, 1);
        ctu::hlld_fan<0, double>(L + 9 * i, R + 9 * i, J + 9 * i, s, gam, 1.0, 1);
        long double l[9], r[9], f[9], sl;
        for (int q = 0; q < 9; q++) { l[q] = L[9 * i + q]; r[q] = R[9 * i + q]; f[q] = 0; }
        ctu::hlld_fan<0, long double>(l, r, f, sl, (long double)gam, 1.0L, 1);
        for (int q = 0; q < 9; q++) {
            hi[9 * i + q] = (double)f[q];
            lo[9 * i + q] = (double)(f[q] - (long double)hi[9 * i + q]);
        }
    }
}
}
"""


@pytest.fixture(scope="module")
def dev(tmp_path_factory):
    d = tmp_path_factory.mktemp("device_math")
    os.makedirs(d / "hip")
    (d / "hip" / "hip_runtime.h").write_text("")
    (d / "t.cpp").write_text(SHIM)
    out = str(d / "t.so")
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-ffp-contract=off", "-Wno-attributes", "-fPIC", "-shared", "-I",
                           str(d), "-I", CSRC, "-o", out, str(d / "t.cpp"), "-lm"])
    return C.CDLL(out)


def call(f, *a):
    a = [np.ascontiguousarray(x, dtype=np.float64) for x in a]
    r = np.empty_like(a[0])
    p = [x.ctypes.data_as(C.POINTER(C.c_double)) for x in (*a, r)]
    f(C.c_int(a[0].size), *p)
    return r


SPECIAL = np.array([0.0, -0.0, np.inf, -np.inf, np.nan])


def operands():
    rng = np.random.default_rng(5)
    return np.concatenate([rng.uniform(1.0, 2.0, 20000) * np.exp2(rng.integers(-500, 500, 20000)),
                           rng.uniform(1.0, 2.0, 2000) * np.exp2(rng.integers(-1000, 1000, 2000))])


def ulps(got, ref):
    return np.abs(got - ref) / np.spacing(np.abs(ref))


def test_operators_round_as_the_languages_within_an_ulp(dev):
    x = operands()
    y = x[::-1].copy() * np.where(np.arange(x.size) % 2, 1.0, -1.0)
    ok = (np.abs(np.log2(x)) + np.abs(np.log2(np.abs(y)))) < 1000
    assert ulps(call(dev.t_rcp, y), 1.0 / y).max() <= 1.0
    assert ulps(call(dev.t_root, x), np.sqrt(x)).max() <= 1.0
    assert ulps(call(dev.t_quot, x[ok], y[ok]), x[ok] / y[ok]).max() <= 1.0
    # two roundings in 1 / sqrt(x): 1.5 ulp from it at most
    assert ulps(call(dev.t_rsq, x), 1.0 / np.sqrt(x)).max() <= 2.0


def test_operators_at_zero_infinity_and_nan(dev):
    s = SPECIAL
    with np.errstate(all="ignore"):
        assert np.array_equal(call(dev.t_rcp, s), 1.0 / s, equal_nan=True)
        assert np.array_equal(np.signbit(call(dev.t_rcp, s[:4])), np.signbit(1.0 / s[:4]))
        assert np.array_equal(call(dev.t_root, s), np.sqrt(s), equal_nan=True)
        assert np.isnan(call(dev.t_root, [-1.0])).all()
        a, b = (v.reshape(-1) for v in np.meshgrid(np.append(s, [2.0, -3.0]), np.append(s, [2.0, -3.0])))
        assert np.array_equal(call(dev.t_quot, a, b), a / b, equal_nan=True)
    # the reciprocal root is for positive finite arguments: NaN elsewhere
    assert np.isnan(call(dev.t_rsq, np.append(s, -1.0))).all()


def mc_selects(dp, dm):
    """the monotonised central limiter by its sign test"""
    c = 0.5 * (dp + dm)
    m = np.fmin(np.fmin(np.abs(c), 2.0 * np.abs(dp)), 2.0 * np.abs(dm))
    return np.where(dp * dm > 0.0, np.copysign(m, c), 0.0)


def test_mc_limiter_is_flat_next_to_nan(dev):
    rng = np.random.default_rng(3)
    v = np.concatenate([SPECIAL, [1.0, -1.0, 3.0, -3.0, 1e-170, -1e-170, 5e-324], rng.standard_normal(200)])
    dp, dm = (x.reshape(-1) for x in np.meshgrid(v, v))
    with np.errstate(all="ignore"):
        ref = mc_selects(dp, dm)
    got = call(dev.t_mc, dp, dm)
    assert np.array_equal(got, ref)
    assert (got[np.isnan(dp) | np.isnan(dm)] == 0.0).all()


def states(n, dv, seed):
    """pairs of neighbouring states that differ by about dv"""
    rng = np.random.default_rng(seed)
    V = np.zeros((n, 9))
    V[:, 0] = rng.uniform(0.6, 1.6, n)
    V[:, 4] = rng.uniform(0.4, 0.9, n)
    V[:, 1:4] = 0.5 * rng.standard_normal((n, 3))
    V[:, 5:8] = 0.6 * rng.standard_normal((n, 3))
    W = V * (1.0 + dv * rng.standard_normal(V.shape))
    W[:, 5] = V[:, 5]
    return V, W


@pytest.mark.parametrize("dv", [1e-6, 1e-3, 1e-2, 0.1])
def test_hlld_rounds_no_more_than_the_jump_form(dev, dv):
    """FP64 HLLD takes the physical flux of the state at the interface; its
    rounding error, row by row, is no larger than that of F_k + S_k (U*_k -
    U_k) (20000 faces: the ratio of two mean errors is good to 2 %)."""
    V, W = states(20000, dv, 17)
    n = len(V)
    out = [np.zeros((n, 9)) for _ in range(4)]
    p = [x.ctypes.data_as(C.POINTER(C.c_double)) for x in (V, W)] + [C.c_double(5.0 / 3.0)]
    p += [x.ctypes.data_as(C.POINTER(C.c_double)) for x in out]
    dev.t_hlld(C.c_int(n), *p)
    F, J, hi, lo = out
    eF, eJ = (np.abs((x - hi) - lo).mean(0) for x in (F, J))
    for q in (0, 1, 2, 3, 4, 6, 7):
        assert eF[q] <= 1.02 * eJ[q], (q, eF[q] / eJ[q])
