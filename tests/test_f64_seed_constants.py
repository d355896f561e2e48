"""The polynomial constants of the FP64 seeds are what the comment beside them says (CPU): sincospi_seed64 in
csrc/kernels_f64.hip sums the Taylor series of sin(pi f) and cos(pi f), coefficients (-1)^k pi^j / j! rounded to FP64, and
the first term left out is below 2^-58 of the result on |f| <= 1/4."""
import os
import re
from fractions import Fraction
from math import factorial

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
# pi to 50 digits
PI = Fraction(31415926535897932384626433832795028841971693993751, 10**49)


def literals(body, name):
    first = re.search(rf"[ ,]{name} = ([-+.\de]+)", body).group(1)
    return [float(first)] + [float(v) for v in re.findall(rf" {name} = fma\({name}, x, ([-+.\de]+)\)", body)]


def test_seed_coefficients_are_the_taylor_series():
    src = open(os.path.join(ROOT, "paper_2307_12041_amd", "csrc", "kernels_f64.hip")).read()
    body = src[src.index("void sincospi_seed64("):]
    body = body[:body.index("\n}\n")]
    sin, cos = literals(body, "p"), literals(body, "r")
    assert len(sin) == 9 and len(cos) == 9
    for got, j0 in ((sin, 1), (cos, 0)):
        want = [float((-1)**k * PI**(2 * k + j0) / factorial(2 * k + j0)) for k in range(9)]
        assert got[::-1] == want, (got[::-1], want)
    quarter = Fraction(1, 4)
    assert PI**19 / factorial(19) * quarter**19 / (PI * quarter * Fraction(9, 10)) < Fraction(1, 2**58)   # sin(pi/4) > 0.9 pi/4
    assert PI**18 / factorial(18) * quarter**18 / Fraction(7, 10) < Fraction(1, 2**58)                    # cos(pi/4) > 0.7
