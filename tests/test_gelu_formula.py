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
    """max(z, 0) - |z| 2^p(a) with a = min(|z|, held): the tail beyond the range of the fit, large arguments, infinities and NaN."""
    text = open(SOURCE).read().split("inline float gelu_wide", 1)[1].split("}", 1)[0]
    c = [np.float32(v) for v in re.findall(r"(?:p = |p, a, )(-?[0-9.e+-]+)f", text)]
    held = np.float32(re.search(r"fminf\(__builtin_fabsf\(z\), ([0-9.]+)f\)", text).group(1))
    assert "return fmaf(-__builtin_fabsf(z), __builtin_amdgcn_exp2f(p), __builtin_fmaxf(z, 0.f));" in text

    def gelu(z):
        a = np.minimum(np.abs(z), held).astype(np.float64)
        p = np.full_like(z, c[0])
        for k in c[1:]:
            p = (p.astype(np.float64) * a + k).astype(np.float32)
        with np.errstate(invalid="ignore"):
            return (np.maximum(z, 0) - np.abs(z).astype(np.float64) * np.exp2(p.astype(np.float64)).astype(np.float32)).astype(np.float32)

    z = np.concatenate([np.linspace(-200, -4, 200001), np.linspace(4, 200, 200001)]).astype(np.float32)
    exact = z.astype(np.float64) * torch.special.ndtr(torch.from_numpy(z.astype(np.float64))).numpy()
    error = np.abs(gelu(z) - exact)
    assert (error[z < 0].max() < 9e-6 and error[z < -5.5].max() < 1.2e-7 and (error[z > 0] < 9e-6 + 6e-8 * z[z > 0]).all())
    np.testing.assert_allclose(gelu(np.array([-65504, -1e10, 65504, 3e38], np.float32)), [0, 0, 65504, 3e38], atol=1e-12, rtol=1e-7)
    assert not np.isfinite(gelu(np.array([-np.inf, np.inf, np.nan], np.float32))).any()
