"""Register transforms of the 3/2 grids of 16 ... 256 modes, each size along x and along z, GPU against the
oracle: transforms both ways and a substep (elided fixed-point path, plane batches, and a z grid finer than 3/2,
whose padding is not known at compile time).  Tolerances as the other substep tests'."""
import dataclasses

import numpy as np
import pytest

from oracle.fourier import to_physical, to_spectral
from paper_2206_09878_amd.workloads import make_inputs, workload
from tests.test_gpu_parity import TOL, check_pair, gplan, gpu_substep, hermitian, host, oracle_substep, rel, spread_tolerances

pytestmark = pytest.mark.gpu


def grid(n1, n2, n3, m3=None):
    return dataclasses.replace(workload("small", n=n1, n2=n2), n3=n3, m3=m3 or 3 * n3 // 2)


# (x modes, z modes, z points, planes per batch); transform lengths are 3/2 of the modes
CASES = [(16, 24, 0, 0), (24, 16, 0, 0), (24, 36, 0, 5), (36, 72, 0, 0), (72, 36, 0, 0), (108, 16, 0, 0), (16, 108, 0, 0),
         (144, 16, 0, 0), (16, 144, 0, 4), (192, 24, 0, 0), (24, 192, 0, 0), (216, 16, 0, 0), (16, 216, 0, 0),
         (256, 16, 0, 0), (16, 256, 0, 0), (16, 20, 36, 0), (36, 64, 108, 0), (24, 100, 162, 0)]


@pytest.mark.parametrize("n1,n3,m3,pb", CASES)
def test_sizes(n1, n3, m3, pb):
    w = grid(n1, 12, n3, m3)
    print("sizes", (w.n1, w.n2, w.n3), (w.m1, w.m3), "planes per batch", pb, flush=True)
    p = gplan(w)
    rng = np.random.default_rng(12)
    V = hermitian(rng, w.shape)
    assert rel(host(p.to_physical(p.to_dev(V))), to_physical(V, w.m1, w.m3)) < TOL
    u = rng.standard_normal((w.n2, w.m3, w.m1))
    assert rel(host(p.to_spectral(p.to_dev(u))), to_spectral(u, w.n1, w.n3)) < TOL
    inp = make_inputs(w, seed=93, stage=1)
    ref = oracle_substep(w, 1, inp)
    check_pair(gpu_substep(w, 1, inp, plane_batch=pb), ref, tols=spread_tolerances(w, 1, ref, inp))
