"""Entries that an operator does not read (the wall values of the Dirichlet and Neumann projections, the plane means
of fields whose (0,0) mode is held apart) may hold anything: NaN and infinity there leave the results the same, bit
for bit, at row counts with and without a remainder of 16."""
import dataclasses

import numpy as np
import pytest

from paper_2206_09878_amd.workloads import workload
from tests.test_gpu_parity import gplan, hermitian

pytestmark = pytest.mark.gpu


def plan_and_fields(n2, seeds):
    w = dataclasses.replace(workload("small", n=16, n2=n2), n3=12, m3=18)
    print("non-finite", (w.n1, w.n2, w.n3), flush=True)
    p = gplan(w)
    star = lambda i: w.shape_star if i == 1 else w.shape  # noqa: E731
    return p, [p.to_dev(hermitian(np.random.default_rng(s), star(i))) for i, s in enumerate(seeds)]


@pytest.mark.parametrize("bad", [float("nan"), float("inf")])
@pytest.mark.parametrize("kind", [1, 2])
@pytest.mark.parametrize("n2", [10, 12, 16, 17, 33, 47])
def test_replaced_wall_values(n2, kind, bad):
    import torch
    p, (v,) = plan_and_fields(n2, [7])
    want = p.project(kind, v)
    v[0], v[-1] = complex(bad, bad), complex(bad, bad)
    got = p.project(kind, v)
    assert torch.isfinite(torch.view_as_real(want)).all()
    assert torch.equal(got, want)


@pytest.mark.parametrize("bad", [float("nan"), float("inf")])
@pytest.mark.parametrize("n2", [10, 16, 33])
def test_plane_means_outside_the_maps(n2, bad):
    """The (0,0) modes of phi2 and Omega2 do not enter m^d, nor those of the cotangents of m1 and m3 the transpose of
    m^c; in the transpose of m^d they reach the plane means alone."""
    import torch
    p, y = plan_and_fields(n2, [8, 9, 10])
    phi, om = (y[0].clone(), y[2].clone())
    m1bar, m3bar = (torch.linspace(a, 1.0, n2, dtype=torch.float64, device="cuda") for a in (0.0, 2.0))
    want = [p.md(phi, om, m1bar, m3bar), p.md_adjoint(*y)[:2], [p.mc_adjoint(*y)]]
    for t in (phi, om, y[0], y[2]):
        t[:, 0, 0] = complex(bad, bad)
    got = [p.md(phi, om, m1bar, m3bar), p.md_adjoint(*y)[:2], [p.mc_adjoint(*y)]]
    for a, b in zip(got, want):
        for s, t in zip(a, b):
            assert torch.isfinite(torch.view_as_real(t)).all()
            assert torch.equal(s, t)
