"""CPU pin of a claim the ConvFFN kernels' comments make: the power of two of a polynomial by which they
evaluate GELU (csrc/esc_gelu.hpp), in float32 in the kernels' order of operations, stays within 2^-21 and 1.2e-7 |v|
of the erf definition (3.4e-7 and 8.1e-8 |v| as it comes out).  The first test is for the comparison that comment
makes: the rational approximation of erf 7.1.26 of Abramowitz and Stegun's handbook, which no kernel evaluates, is held to
6e-7 and 3e-7 |v|.  tests/test_gpu_ffn.py measures the kernels themselves."""
import math

import numpy as np


def test_rational_erf_keeps_gelu_within_its_stated_error():
    f = np.float32
    v = np.linspace(-12.0, 12.0, 600001).astype(f)
    a = np.abs(v) * f(0.70710678118654752440)
    t = (f(1) / (f(0.3275911) * a + f(1))).astype(f)
    q = f(1.061405429) * t + f(-1.453152027)
    for c in (1.421413741, -0.284496736, 0.254829592):
        q = (q * t + f(c)).astype(f)
    e = np.exp2((a * a * f(-1.44269504088896340736)).astype(f)).astype(f)
    erf_a = (f(1) - (q * t).astype(f) * e).astype(f)
    h = f(0.5) * v
    g = (np.abs(h) * erf_a + h).astype(np.float64)
    ref = np.array([0.5 * x * (1.0 + math.erf(x / math.sqrt(2.0))) for x in v.astype(np.float64)])
    err = np.abs(g - ref)
    assert err.max() <= 6e-7, err.max()
    assert (err <= 3e-7 * np.maximum(np.abs(v), 1e-2)).all()
    assert g[np.abs(v) == 0].tolist() == [0.0] * int((v == 0).sum())


def test_power_of_two_form_keeps_gelu_within_its_stated_error():
    # the form the kernels evaluate (csrc/esc_gelu.hpp): h + |h| (1 - 2^-(|v| P(|v|))), h = v / 2.  Bars: relative to |v|
    # the fit's 1e-8, half a rounding of 1 - e (2^-26), half an ulp of the exponential (2^-25) and the last
    # rounding (2^-24), together 1.2e-7; half an ulp of the largest argument, 2^-21, absolutely; P must not
    # turn down beyond the fitted range.  Infinities as in the definition evaluated in floating point.
    f = np.float32
    v = np.concatenate([np.linspace(-12.0, 12.0, 600001), np.logspace(1, 38, 2000), -np.logspace(1, 38, 2000)]).astype(f)

    def fma(a, b, c):
        return (np.asarray(a, np.float64) * b + c).astype(f)

    def gelu(v):
        t = np.abs(v).astype(np.float64)
        with np.errstate(over="ignore", invalid="ignore"):
            q = fma(f(2.834909764715121e-06), t, np.float64(f(-3.937766086892225e-05)))
            for c in (0.0001861801283666864, 0.0001369366073049605, -0.0070634204894304276, 0.052496179938316345,
                      0.4592081904411316, 1.1511051654815674):
                q = fma(q, t, np.float64(f(c)))
            e = np.exp2((-q * t).astype(f).astype(np.float64)).astype(f)
            h = f(0.5) * v
            return fma(np.abs(h), (f(1) - e).astype(np.float64), h.astype(np.float64))

    g, t = gelu(v).astype(np.float64), np.abs(v).astype(np.float64)
    ref = np.array([0.5 * x * math.erfc(-x / math.sqrt(2.0)) for x in v.astype(np.float64)])
    err = np.abs(g - ref)
    assert err[t <= 12].max() <= 2.0 ** -21, err[t <= 12].max()
    assert (err <= 1.2e-7 * np.maximum(t, 1e-2)).all()
    assert g[t == 0].tolist() == [0.0] * int((t == 0).sum())
    special = gelu(np.array([np.inf, -np.inf, np.nan], f))
    assert np.isposinf(special[0]) and np.isnan(special[1]) and np.isnan(special[2])
