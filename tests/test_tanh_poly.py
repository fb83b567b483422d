"""The constants of the fp32 gate's tanh for small arguments (host logic, no GPU): the fit script beside the kernel
reproduces them, their relative error is what the kernel's comment says, and a float32 evaluation in the kernel's order
stays within one unit in the last place."""
import importlib.util
import os
import re

import numpy as np

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2509_21354_amd", "csrc")


def _fit_module():
    spec = importlib.util.spec_from_file_location("fit_tanh_poly", os.path.join(CSRC, "fit_tanh_poly.py"))
    m = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(m)
    return m


def test_kernel_constants_are_the_fit_and_accurate():
    m = _fit_module()
    src = open(os.path.join(CSRC, "lstm_generic.hip")).read()
    line = re.search(r"const float p = fmaf\(fmaf\(fmaf\(fmaf\((.*)\);", src).group(1)
    kernel = np.array([float(v) for v in re.findall(r"(-?\d\.\d+)f", line)][::-1])        # c0 .. c4
    assert len(kernel) == m.DEGREE and abs(float(re.search(r"kTanhSmall = ([0-9.]+)f", src).group(1)) - m.X_MAX) < 1e-9
    assert np.allclose(kernel, m.coefficients(), rtol=5e-6, atol=0)
    x = np.linspace(1e-4, m.X_MAX, 200001)
    assert np.abs(m.relative_error(x, kernel)).max() < 1.4e-9
    x = x.astype(np.float32)
    want = np.tanh(x.astype(np.float64))
    assert (np.abs(m.tanh_f32(x, kernel) - want) <= np.spacing(want.astype(np.float32))).all()
