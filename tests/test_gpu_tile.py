"""Column kernels on LDS tiles (32, 16 or 8 columns per tile, the widest whose rows fit), GPU against the oracle:
row counts on both sides of every change of the tile width and of the streaming kernels' takeover, rows one
over and under a block of 16, column counts that leave the last tile ragged, and orders below the widest.
Tolerances: 1e-11, or the spread of the oracle's own results under other roundings where that is larger
(spread_tolerances)."""
import dataclasses

import numpy as np
import pytest

from oracle.lmvd import Plan as OPlan, curl_free_momentum, divergence_free_momentum
from paper_2206_09878_amd.workloads import make_inputs, workload
from tests.conftest import oracle_config
from tests.test_gpu_parity import (check_pair, dense_solves_in_oracle, gplan, gpu_substep, hermitian, host, oracle_substep, rel,
                                   spread_tolerances)

pytestmark = pytest.mark.gpu


# tile width changes: m^c and prologue after 191 and 383 rows, right-hand sides 64, 143 and 256 (then streaming),
# projections 256; on these 88 columns a single instance takes 16 columns where a graph takes 32
CASES = [(n2, 8, s) for n2, s in ((11, 0), (15, 1), (16, 0), (17, 1), (31, 0), (64, 1), (65, 0), (127, 0), (128, 1),
                                  (144, 0), (145, 1), (191, 0), (192, 0), (256, 1), (257, 0), (288, 0), (384, 0))]
CASES += [(33, 6, 0), (64, 5, 1), (40, 7, 1)]


@pytest.mark.parametrize("n2,order,stage", CASES)
def test_tile_rows(n2, order, stage):
    w = dataclasses.replace(workload("small", n=16, n2=n2), order=order)
    w = dataclasses.replace(w, n3=12, m3=18)
    print("tiles", (w.n1, w.n2, w.n3), "order", order, "stage", stage, flush=True)
    inp = make_inputs(w, seed=91, stage=stage)
    ref = oracle_substep(w, stage, inp)
    check_pair(gpu_substep(w, stage, inp), ref, tols=spread_tolerances(w, stage, ref, inp))


# (tile width changes of the transposed solves after 111 and 255 rows, of m^c from coefficients 191: test_gpu_routes.py)
@pytest.mark.parametrize("n2,order", [(11, 8), (16, 8), (17, 8), (111, 8), (112, 8), (223, 8), (224, 8), (271, 8), (272, 8),
                                      (33, 6), (64, 5)])
def test_tile_operators(n2, order):
    """m^d, m^c and the transposes of both and of the projections.  The maps against the oracle's (1e-11, or four times
    what dense pivoted solves change in the oracle), the transposes by dot products with the maps, to the same accuracy."""
    import torch
    w = dataclasses.replace(workload("small", n=16, n2=n2), order=order)
    w = dataclasses.replace(w, n3=12, m3=18)
    print("operators", (w.n1, w.n2, w.n3), "order", order, flush=True)
    p = gplan(w)
    op = OPlan(oracle_config(w))
    inp = make_inputs(w, seed=92)
    rhot = hermitian(np.random.default_rng(5), w.shape)
    md_in = [inp[k] for k in ("phi2", "omega2", "m1bar", "m3bar")]
    maps = lambda: (divergence_free_momentum(op, *md_in), curl_free_momentum(op, rhot)[:3])
    ref = maps()
    with dense_solves_in_oracle():
        alt = maps()
    dev = [p.to_dev(x) for x in md_in]
    got = p.md(*dev), p.mc(p.to_dev(rhot))
    tol = []
    for g, r, a in zip(got, ref, alt):
        tol.append(max([1e-11] + [4.0 * rel(y, x) for x, y in zip(r, a)]))
        for x, y in zip(g, r):
            assert rel(host(x), y) < tol[-1]

    def dot(a, b):
        return torch.sum(torch.view_as_real(a) * torch.view_as_real(b)).item() if a.is_complex() else torch.sum(a * b).item()

    def check(xs, ys, xts, bar):  # <A x, y> = <x, A^T y>, ys the pairs (A x, y)
        lhs, rhs = sum(dot(a, b) for a, b in ys), sum(dot(a, b) for a, b in zip(xs, xts))
        assert abs(lhs - rhs) < bar * sum(a.norm().item() * b.norm().item() for a, b in ys)

    y = [p.to_dev(hermitian(np.random.default_rng(6 + i), w.shape_star if i == 1 else w.shape)) for i in range(3)]
    check(dev, list(zip(got[0], y)), p.md_adjoint(*y), tol[0])
    check([p.to_dev(rhot)], list(zip(got[1], y)), [p.mc_adjoint(*y)], tol[1])
    for kind in range(3):
        v = p.to_dev(rhot)
        check([v], [(p.project(kind, v), y[0])], [p.project_adjoint(kind, y[0])], 1e-11)


@pytest.mark.parametrize("n2s", [(11, 16, 33), (64, 65, 96), (127, 128, 129), (143, 144, 191), (192, 383, 384)])
def test_tile_widths_agree(n2s):
    """A graph's grouped launches run the widest tiles that fit, a small instance alone narrower ones, with Omega2 in
    rows of its own or after c: bit for bit the same, over both stages."""
    import torch
    from paper_2206_09878_amd.lmvd import GraphBatch, Stepper
    from tests.test_gpu_graph import state_tensors
    ws = [dataclasses.replace(workload("small", n=16, n2=n2), n3=12, m3=18) for n2 in n2s]
    A, B = ([Stepper(gplan(w), make_inputs(w, seed=94, stage=0), stage=0) for w in ws] for _ in range(2))
    print("widths", n2s, flush=True)
    g = GraphBatch(A, nsub=4)
    assert g.grouped
    for _ in range(2):
        g.launch()
        for s in B:
            for _ in range(4):
                s.substep()
        torch.cuda.synchronize()
        for a, b in zip(A, B):
            for x, y in zip(state_tensors(a), state_tensors(b)):
                assert torch.equal(x, y)
