"""The centred phase factors of the regular fill in double (the phase of
R - |d| by short polynomials, e^{-jkR} of Sec. II-B): the coefficients and the
bounds of their range are read from the kernel source, and the error of the
fits over that range has to stay within that of the nine-term fits that the
reduced phases take over a quarter turn, 3.3e-19 and 2.6e-20 for sine and
cosine (interpolation error of sin(2 pi sqrt u) / sqrt u and (cos(2 pi sqrt u)
- 1) / u at nine Chebyshev nodes, evaluated in 60 digits); the loss factor's
Taylor polynomial within a hundredth of a rounding."""
import os
import re
from decimal import Decimal, getcontext

getcontext().prec = 60
SRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2111_11058_amd", "csrc", "fill.hip")
PI = Decimal("3.14159265358979323846264338327950288419716939937510582097494459")


def _series(x, first, k):
    """sin (first = x, k = 1) or cos (first = 1, k = 0)."""
    t = s = first
    while abs(t) > Decimal(10) ** -55:
        t = -t * x * x / ((k + 1) * (k + 2))
        s, k = s + t, k + 2
    return s


def _source():
    src = open(SRC).read()
    num = lambda t: [Decimal(x) for x in re.findall(r"-?\d+\.\d+(?:e-?\d+)?", t)]  # noqa: E731
    sn, cs = (num(re.search(r"%s\[8\] = \{(.*?)\}" % n, src, re.S).group(1)) for n in ("kSinC", "kCosC"))
    a, b = (num(re.search(r"constexpr double %s = (.*?);" % n, src).group(1)) for n in ("kCentredRev", "kCentredExp"))
    assert len(sn) == 8 and len(cs) == 8
    return sn, cs, a[0] / a[1], b[0] / b[1]


def test_fits_over_their_range():
    sn, cs, rev, _ = _source()
    es = ec = Decimal(0)
    for i in range(1, 301):
        x = rev * i / 300
        u = x * x
        s = x * sum(c * u ** j for j, c in enumerate(sn))
        c = 1 + u * sum(v * u ** j for j, v in enumerate(cs))
        es = max(es, abs(s - _series(2 * PI * x, 2 * PI * x, 1)))
        ec = max(ec, abs(c - _series(2 * PI * x, Decimal(1), 0)))
    assert es <= Decimal("3.3e-19") and ec <= Decimal("2.6e-20"), (es, ec)


def test_loss_polynomial():
    b = _source()[3]
    t, s = Decimal(1), Decimal(1)
    for k in range(1, 9):
        t = -t * b / k
        s += t
    assert abs(s - (-b).exp()) <= Decimal("0.01") * Decimal(2) ** -53
