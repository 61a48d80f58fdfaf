"""GELU of the kernels for many tokens: max(z, 0) - a 2^p(a) with a = min(|z|, 5.5), the coefficients read from the kernels' source."""
import os
import re

import numpy as np
import torch

SOURCE = os.path.join(os.path.dirname(__file__), "..", "paper_2207_05022_amd", "csrc", "gemm_tile.hpp")


def test_error_of_the_many_token_gelu():
    text = open(SOURCE).read().split("inline float gelu_wide", 1)[1].split("}", 1)[0]
    c = [np.float32(v) for v in re.findall(r"(?:p = |p, a, )(-?[0-9.e+-]+)f", text)]
    assert len(c) == 5
    z = np.concatenate([np.linspace(-12, 12, 400001), np.logspace(-8, 0, 2000), -np.logspace(-8, 0, 2000), [65504, -65504, 3e38, -3e38]]).astype(np.float32)
    a = np.minimum(np.abs(z), np.float32(5.5)).astype(np.float64)
    p = np.full_like(z, c[0])
    for k in c[1:]:
        p = (p.astype(np.float64) * a + k).astype(np.float32)      # (a fused multiply-add rounds once)
    y = (np.maximum(z, 0) - a * np.exp2(p.astype(np.float64)).astype(np.float32)).astype(np.float32).astype(np.float64)
    z = z.astype(np.float64)
    want = z * torch.special.ndtr(torch.from_numpy(z)).numpy()
    error = np.abs(y - want)
    small = np.abs(z) <= 12
    assert error[small].max() < 9e-6
    np.testing.assert_allclose(y[~small], want[~small], atol=1e-6)
    relative = error / np.maximum(np.abs(want), 1e-30)
    assert relative[small & (z > -1)].max() < 1e-4 and relative[small & (z > -3)].max() < 2e-3


def test_many_token_gelu_far_out_and_where_there_is_no_number():
    """max(z, none) - a 2^p(a) with none = 0 max|z| over eight values: the bits of max(z, 0) - a 2^p(a) where all of them are numbers, far beyond the
    range of the fit, too; infinities and NaN come out as themselves."""
    source = open(SOURCE).read()
    text = source.split("inline float gelu_wide", 1)[1].split("}", 1)[0]
    c = [np.float32(v) for v in re.findall(r"(?:p = |p, a, )(-?[0-9.e+-]+)f", text)]
    assert "fminf(__builtin_fabsf(z), 5.5f)" in text
    assert "return fmaf(-a, __builtin_amdgcn_exp2f(p), __builtin_fmaxf(z, none));" in text
    assert "most = __builtin_elementwise_maximum(most, __builtin_fabsf(z[e]))" in source and "return most * 0.f;" in source

    def gelu(z, positive):
        a = np.fmin(np.abs(z), np.float32(5.5)).astype(np.float64)
        p = np.full_like(z, c[0])
        for k in c[1:]:
            p = (p.astype(np.float64) * a + k).astype(np.float32)
        return (positive - a * np.exp2(p.astype(np.float64)).astype(np.float32)).astype(np.float32)

    def part(z):
        with np.errstate(invalid="ignore"):
            return np.fmax(z, np.maximum.reduce(np.abs(z).reshape(-1, 8), axis=1).repeat(8) * np.float32(0.0))     # (np.maximum: NaN stays)

    z = np.concatenate([np.linspace(-200, 200, 400000), np.logspace(-44, 38, 4000), -np.logspace(-44, 38, 4000)]).astype(np.float32)
    np.testing.assert_array_equal(gelu(z, part(z)), gelu(z, np.maximum(z, 0)))
    far = np.abs(z) > 5.5
    np.testing.assert_allclose(gelu(z, part(z))[far], np.maximum(z, 0)[far], atol=1.5e-7, rtol=6e-8)
    for odd in (-np.inf, np.inf, np.nan):
        for at in range(8):
            eight = np.linspace(-7, 7, 8, dtype=np.float32)
            eight[at] = odd
            np.testing.assert_array_equal(gelu(eight, part(eight))[at], np.float32(odd))
