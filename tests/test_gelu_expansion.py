"""The expansion of the normal distribution function that the fused GELU epilogues use, from its coefficients in the source."""
import os
import re

import numpy as np
from scipy.special import erfcx

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_normal_cdf_coefficients():
    """Phi(-|u|) = exp(-u^2 / 2) w: w of the source's fp32 coefficients, evaluated in 64 bits, against erfcx(|u| / sqrt 2) / 2."""
    src = open(os.path.join(ROOT, "paper_2605_18750_amd", "csrc", "gemm_mfma.hip")).read()
    body = src[src.index("float normal_cdf("):]
    body = body[:body.index("\n}")]
    scale = np.float64(np.float32(re.search(r"\* ([0-9.]+)f, t = ", body).group(1)))
    coef = [np.float64(np.float32(v)) for v in re.findall(r"float r = (-?[0-9.]+)f|fmaf\(r, s, (-?[0-9.]+)f\);", body) for v in v if v]
    assert len(coef) == 9 and "fmaf(r, s, 0.5f) * e" in body
    for lo, hi, bound in ((0, 1, 5e-8), (1, 3, 2e-7), (3, 6, 5e-7), (6, 13, 1.7e-6)):
        u = np.linspace(lo, hi, 100001)
        x = u * scale
        w = np.polyval(coef + [0.5], -x / (1 + x))
        err = np.abs(w / (0.5 * erfcx(u / np.sqrt(2))) - 1).max()
        assert err <= bound, (lo, hi, err)
