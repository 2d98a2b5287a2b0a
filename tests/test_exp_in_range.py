"""exp_in_range() of the kernels, evaluated here with the coefficients of the source: below one unit in the last place."""
import re

import numpy as np

from paper_2505_23949_amd import build


def _fma(a, b, c):
    # (80-bit numbers: the product is off by 2^-64 of itself where a fused one is exact)
    return (np.longdouble(1) * a * b + c).astype(np.float64)


def test_error_below_one_ulp():
    source = (build.CSRC / "dykstra_sort.hpp").read_text()
    body = source[source.index("double exp_in_range(double x)"):]
    body = body[:body.index("ldexp")]
    constants = {k: float.fromhex(v) for k, v in re.findall(r"(k\w+) = (0x[0-9a-fp.+-]+)", body)}
    first = float.fromhex(re.search(r"double q = (0x[0-9a-fp.+-]+);", body).group(1))
    rest = re.findall(r"q = fma\(q, r, (0x[0-9a-fp.+-]+|1\.0)\);", body)
    assert len(constants) == 4 and len(rest) == 11
    rng = np.random.default_rng(1)
    x = np.concatenate([rng.uniform(-708, 0, 200000), rng.uniform(-83, 55, 50000), rng.uniform(-1, 1, 50000), -np.logspace(-12, 0, 5000),
                        np.arange(-1021, 80) * np.log(2.0), (np.arange(-1021, 80) + 0.5) * np.log(2.0), [0.0, -700.0, -83.0, 55.0]])
    n = _fma(x, constants["kLog2e"], constants["kRound"]) - constants["kRound"]
    r = _fma(n, -constants["kLn2Lo"], _fma(n, -constants["kLn2Hi"], x))
    q = np.full_like(x, first)
    for c in rest:
        q = _fma(q, r, float.fromhex(c) if c != "1.0" else 1.0)
    got, want = np.ldexp(q, n.astype(int)), np.exp(x.astype(np.longdouble))
    ulp = np.spacing(want.astype(np.float64)).astype(np.longdouble)
    error = np.abs((got - want) / ulp)
    assert error.max() < 1.0, (error.max(), x[error.argmax()])
