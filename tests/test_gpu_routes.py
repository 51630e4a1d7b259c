"""Every route of the column kernels and of the transforms, GPU against the oracle.

  * Operators and their transposes on tiles of 32 columns (grids with more than 16 columns for every compute unit), on
    pair tiles whose last one is ragged, at the edges where the transposed solves (111, 255, 559 rows), m^c from
    coefficients and m^d (191, 383) and the projections (256, 432) change their tiles, and streaming: beyond 592 rows a
    plan has no tiles, and 593 to 600 rows end the streaming sweeps, unrolled by 4 and 8, in each of their tails.
  * Substeps on the streaming kernels at 593 to 599 and at 9 and 10 rows, every second one with laws that depend on z;
    with such laws at the edges of the strain (96, 208, 416 rows) and right-hand sides (143, 256).
  * The transforms of sizes without register plans, along either axis and both, with plane batches and laws.

Tolerances: 1e-11, or four times what other roundings and eliminations change in the oracle (the maps by dense pivoted
solves, substeps by spread_tolerances); the transposes by dot products with the maps, to the same accuracy."""
import dataclasses

import numpy as np
import pytest

import tests.test_gpu_adjoint as transposes
import tests.test_gpu_substep_adjoint as adjoints
from oracle.fourier import to_physical, to_spectral
from oracle.lmvd import Plan as OPlan, curl_free_momentum, divergence_free_momentum
from paper_2206_09878_amd.workloads import make_inputs, workload
from tests.conftest import oracle_config
from tests.test_gpu_parity import (TOL, check_pair, dense_solves_in_oracle, gplan, gpu_substep, hermitian, host, oracle_substep,
                                   rel, spread_tolerances)
from tests.test_gpu_transport import with_laws

pytestmark = pytest.mark.gpu


def grid(n1, n2, n3, order=8):
    return dataclasses.replace(workload("small", n=n1, n2=n2), n3=n3, m3=3 * n3 // 2, order=order)


OPERATORS = [(108, 17, 108, 8), (108, 33, 108, 8), (96, 64, 128, 6), (36, 17, 36, 8), (36, 65, 36, 8)]
OPERATORS += [(12, n2, 18, 8) for n2 in (12, 111, 112, 191, 192, 255, 256, 257, 383, 384, 432, 433, 559, 560, 592)]
OPERATORS += [(12, n2, 18, 8) for n2 in range(593, 601)] + [(16, 9, 12, 8), (16, 10, 12, 8), (12, 600, 18, 5)]


@pytest.mark.parametrize("n1,n2,n3,order", OPERATORS)
def test_operators(n1, n2, n3, order):
    import torch
    w = grid(n1, n2, n3, order)
    print("operators", (n1, n2, n3), "order", order, flush=True)
    p, op, inp = gplan(w), OPlan(oracle_config(w)), make_inputs(w, seed=92)
    rhot = hermitian(np.random.default_rng(5), w.shape)
    md_in = [inp[k] for k in ("phi2", "omega2", "m1bar", "m3bar")]
    maps = lambda: (divergence_free_momentum(op, *md_in), curl_free_momentum(op, rhot)[:3])  # noqa: E731
    ref = maps()
    with dense_solves_in_oracle():
        alt = maps()
    dev, rdev = [p.to_dev(x) for x in md_in], p.to_dev(rhot)
    got = p.md(*dev), p.mc(rdev)
    tol = [max([TOL] + [4.0 * rel(y, x) for x, y in zip(r, a)]) for r, a in zip(ref, alt)]
    for g, r, t in zip(got, ref, tol):
        for x, y in zip(g, r):
            assert rel(host(x), y) < t

    def dot(a, b):
        return torch.sum(torch.view_as_real(a) * torch.view_as_real(b)).item() if a.is_complex() else torch.sum(a * b).item()

    def check(xs, ys, xts, bar):  # <A x, y> = <x, A^T y>, ys the pairs (A x, y)
        lhs, rhs = sum(dot(a, b) for a, b in ys), sum(dot(a, b) for a, b in zip(xs, xts))
        assert abs(lhs - rhs) < bar * sum(a.norm().item() * b.norm().item() for a, b in ys)

    y = [p.to_dev(hermitian(np.random.default_rng(6 + i), w.shape_star if i == 1 else w.shape)) for i in range(3)]
    check(dev, list(zip(got[0], y)), p.md_adjoint(*y), tol[0])
    check([rdev], list(zip(got[1], y)), [p.mc_adjoint(*y)], tol[1])
    P = (op.P_plain, op.P_D, op.P_N)
    for kind in range(3):
        b = rhot.reshape(n2, -1).copy()
        if kind:
            b[0] = b[-1] = 0.0
        v = p.project(kind, rdev)
        assert rel(host(v), np.linalg.solve(P[kind], b).reshape(w.shape)) < TOL
        check([rdev], [(v, y[0])], [p.project_adjoint(kind, y[0])], TOL)


STREAMING = [(16, n2, 12, n2 % 4 // 2, n2 % 2) for n2 in (9, 10, *range(593, 600))]
EDGES = [(12, n2, 18, n2 % 2, 1) for n2 in (96, 97, 143, 144, 208, 209, 256, 257, 416, 417)]


@pytest.mark.parametrize("n1,n2,n3,stage,laws", STREAMING + EDGES)
def test_substeps(n1, n2, n3, stage, laws):
    w = with_laws(grid(n1, n2, n3)) if laws else grid(n1, n2, n3)
    print("substep", (n1, n2, n3), "stage", stage, "laws", laws, flush=True)
    inp = make_inputs(w, seed=95, stage=stage)
    ref = oracle_substep(w, stage, inp)
    check_pair(gpu_substep(w, stage, inp), ref, tols=spread_tolerances(w, stage, ref, inp, rounding=True))


@pytest.mark.parametrize("n1,n3,pb,laws", [(12, 12, 0, 0), (12, 12, 5, 1), (12, 16, 0, 1), (16, 12, 0, 1), (16, 18, 4, 0), (12, 18, 0, 1),
                                           (288, 12, 0, 0), (12, 288, 0, 0)])
def test_transforms_without_register_plans(n1, n3, pb, laws):
    w = with_laws(grid(n1, 14, n3)) if laws else grid(n1, 14, n3)
    print("transforms", (w.n1, w.n2, w.n3), (w.m1, w.m3), "planes per batch", pb, "laws", laws, flush=True)
    p, rng = gplan(w), np.random.default_rng(12)
    V = hermitian(rng, w.shape)
    assert rel(host(p.to_physical(p.to_dev(V))), to_physical(V, w.m1, w.m3)) < TOL
    u = rng.standard_normal((w.n2, w.m3, w.m1))
    assert rel(host(p.to_spectral(p.to_dev(u))), to_spectral(u, w.n1, w.n3)) < TOL
    inp = make_inputs(w, seed=96, stage=1)
    ref = oracle_substep(w, 1, inp)
    check_pair(gpu_substep(w, 1, inp, plane_batch=pb), ref, tols=spread_tolerances(w, 1, ref, inp))


def test_transposed_transforms_without_register_plans():
    import torch
    transposes.test_transform_transpose(torch, 12, 25)


@pytest.mark.parametrize("n,n2,stage,guess,kf,pb", [(12, 25, 1, 0, 4, 7), (12, 19, 0, 1, 4, 0), (16, 9, 0, 0, 4, 0), (16, 10, 1, 0, 4, 0)])
def test_adjoint_substep(n, n2, stage, guess, kf, pb):
    """The generic transforms (12 modes) and the streaming column kernels (9 and 10 rows) of the adjoint."""
    adjoints.test_adjoint_against_the_oracle_adjoint(n, n2, stage, guess, kf, pb)
