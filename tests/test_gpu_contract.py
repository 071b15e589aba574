"""The contraction kernels at the edges of their tiles and segments: z3_contract of random
multipoles against the sum written out in FP64, for every number of row tiles, pivot counts
around the groups, segments and launch sizes, and odd leading dimensions."""

import numpy as np
import pytest
import torch

import paper_2408_16847_amd as z3
from tests import gpu_helpers as G

pytestmark = pytest.mark.gpu


def _exact(A, v):
    X = torch.complex(A[:, 0].double(), A[:, 1].double())          # [m+1, nb, P]
    Y = (X * v).contiguous()
    z = torch.stack([Y[m] @ X[m].conj().T.contiguous() for m in range(X.shape[0])])
    s = torch.stack([(X[m].abs() * v.abs()) @ X[m].abs().T.contiguous() for m in range(X.shape[0])])
    return z, s


@pytest.mark.parametrize("prec", ["fp64", "mixed"])
@pytest.mark.parametrize("nb", [1, 8, 9, 16, 20, 32, 33, 64])
@pytest.mark.parametrize("P", [1, 15, 17, 129, 4099])
def test_contract_edges(prec, nb, P):
    G.say("case: contract", prec, nb, P)
    m_max = 3
    g = torch.Generator(device="cuda").manual_seed(1000 * nb + P)
    A = torch.randn((m_max + 1, 2, nb, P), dtype=torch.float64, device="cuda", generator=g)
    A = A if prec == "fp64" else A.float()
    v = torch.randn(P, dtype=torch.float64, device="cuda", generator=g)
    zeta = z3.contract(A, v, m_max, nb, prec=prec)
    got = torch.complex(zeta[..., 0], zeta[..., 1])
    exact, size = _exact(A, v)
    # FP64: every sum of P products, rounded once per addition; mixed: FP32 products and sums
    # over 16 pivots (up to 33 roundings of 6e-8 on each of the two products of a component)
    tol = P * 2.3e-16 + 1e-15 if prec == "fp64" else 66 * 6e-8
    assert torch.all((got - exact).abs() <= tol * size)
    assert torch.equal(got, got.transpose(1, 2).conj())


@pytest.mark.parametrize("prec", ["fp64", "mixed"])
def test_contract_many_segments(prec):
    # more segments than the final reduction takes itself, the last one a few pivots
    G.say("case: contract segments", prec)
    P, nb, m_max = 700_003, 5, 1
    g = torch.Generator(device="cuda").manual_seed(7)
    A = torch.randn((m_max + 1, 2, nb, P), dtype=torch.float64, device="cuda", generator=g)
    A = A if prec == "fp64" else A.float()
    v = torch.rand(P, dtype=torch.float64, device="cuda", generator=g)
    zeta = z3.contract(A, v, m_max, nb, prec=prec)
    again = z3.contract(A, v, m_max, nb, prec=prec)
    assert torch.equal(zeta, again)  # fixed order of the sums
    exact, size = _exact(A, v)
    got = torch.complex(zeta[..., 0], zeta[..., 1])
    # random signs: the rounding of 7e5 additions grows at most linearly
    assert torch.all((got - exact).abs() <= (P * 2.3e-16 if prec == "fp64" else 66 * 6e-8) * size)
