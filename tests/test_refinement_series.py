"""Limits of the Jacobi eigensolver's refinement steps against the series they
truncate (CPU only): W = E + sqrt(I + E^2) for anti-Hermitian E, whose
eigenvalues i x give sqrt(1 - x^2)."""
import os
import re
from decimal import Decimal, getcontext

import pytest

SRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2601_10557_amd", "csrc",
                   "dense.hip")
# sqrt(1 + t) up to t^6
SERIES = ["1", "0.5", "-0.125", "0.0625", "-0.0390625", "0.02734375", "-0.0205078125"]


def limits():
    text = open(SRC).read()
    return {n: Decimal(re.search(r"\b%s = ([0-9.e-]+)" % n, text).group(1))
            for n in ("REFINE_MAX", "REFINE_MID", "REFINE_SHORT")}


@pytest.mark.parametrize("name,terms", [("REFINE_MAX", 7), ("REFINE_MID", 5), ("REFINE_SHORT", 2)])
def test_truncation_is_below_rounding(name, terms):
    getcontext().prec = 50
    x = limits()[name]
    t = -x * x
    series = sum(Decimal(c) * t ** j for j, c in enumerate(SERIES[:terms]))
    assert abs((1 + t).sqrt() - series) <= Decimal(2) ** -53


def test_the_terms_are_those_of_the_square_root():
    getcontext().prec = 80
    t = Decimal("-1e-6")
    exact = (1 + t).sqrt()
    for n in range(1, 8):
        rest = exact - sum(Decimal(c) * t ** j for j, c in enumerate(SERIES[:n]))
        assert abs(rest) < abs(t) ** n


def test_the_kernel_has_these_terms():
    text = open(SRC).read()
    body = text[text.index("void refine_w_kernel"):]
    body = body[:body.index("\n}\n")]
    for c in SERIES[1:]:
        assert c.lstrip("-") in body, c
