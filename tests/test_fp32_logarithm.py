"""The polynomial of the fp32 forward's logarithm (csrc/sb_fwd_f32.hip), its coefficients as they stand in the source, against log1p in 64 bits."""
import os
import re

import numpy as np

from paper_2410_17980_amd import build


def test_polynomial_of_the_logarithm():
    text = open(os.path.join(build.CSRC, "sb_fwd_f32.hip")).read()
    body = re.search(r"float log1p_f32\(float e\)\n\{(.*?)\n\}", text, re.S).group(1)
    coefs = [float(np.float32(c)) for c in re.findall(r"(-?\d\.\d+)f", body)]
    assert len(coefs) == 10
    e = np.linspace(2.0 ** -24, 1.0, 1 << 20)
    assert np.abs((e - e * e * np.polyval(coefs, e)) / np.log1p(e) - 1.0).max() <= 9e-10
