"""Entries that an operator does not read (the wall values of the Dirichlet and Neumann projections) may hold
anything: NaN and infinity there leave the results the same, bit for bit, at row counts with and without a remainder
of 16."""
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
