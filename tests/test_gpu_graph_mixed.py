"""Graphs of instances whose steps run different kernels (with and without register transforms along either axis, plane
batches, laws that depend on z, streaming and tile column kernels): grouped, and over two launches bit for bit the same
as their substeps one by one."""
import dataclasses

import pytest

from paper_2206_09878_amd.workloads import make_inputs, workload
from tests.test_gpu_graph import state_tensors

pytestmark = pytest.mark.gpu


def small(n1, n2, n3, **kw):
    w = workload("small", n=n1, n2=n2)
    return dataclasses.replace(w, n3=n3, m3=3 * n3 // 2, **kw)


VAR = dict(mu_z=(0.2 * 5e-3, 0.0, 0.0))
MIXES = {
    "12 beside 16": [(small(12, 17, 12), 0), (small(16, 17, 16), 0), (small(12, 33, 16), 0), (small(12, 15, 12), 0),
                     (small(24, 17, 16), 0), (small(16, 20, 16), 0)],
    "288 beside 256": [(small(288, 12, 16), 0), (small(256, 12, 16), 0), (small(16, 12, 288), 0)],
    "plane batches": [(small(16, 17, 16), 5), (small(16, 17, 16), 0), (small(12, 17, 12), 4)],
    "laws": [(small(16, 17, 16, **VAR), 0), (small(16, 33, 16), 0), (small(12, 17, 12, **VAR), 0)],
    "rows": [(small(16, 10, 16), 0), (small(16, 17, 16), 0), (small(12, 300, 12), 0)],
}


@pytest.mark.parametrize("mix", sorted(MIXES))
def test_mixed_instances_are_grouped(mix):
    import torch
    from paper_2206_09878_amd.lmvd import GraphBatch, Plan, Stepper
    print("mix", mix, [(w.n1, w.n2, w.n3, w.order, pb) for w, pb in MIXES[mix]], flush=True)
    A, B = ([Stepper(Plan(w, plane_batch=pb), make_inputs(w, seed=80 + i, stage=0), stage=0)
             for i, (w, pb) in enumerate(MIXES[mix])] for _ in range(2))
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
                assert torch.isfinite(torch.view_as_real(x) if x.is_complex() else x).all()
                assert torch.equal(x, y)
