"""What a plan holds on the GPU: the A(k) factors once, in the layout of the kernels that read them."""
import ctypes

import pytest

from paper_2206_09878_amd.workloads import make_inputs, workload
from tests.test_gpu_graph import state_tensors

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,n2,order", [(128, 129, 8), (96, 97, 6)])
def test_factors_are_held_once(n, n2, order):
    """A row of the elimination has 9 entries (order 8; fewer below), 10 with those that fill the tiles' rows: a second
    copy would pass 1.5 times the first's size."""
    import dataclasses
    import torch
    from paper_2206_09878_amd import lmvd
    w = dataclasses.replace(workload("small", n=n, n2=n2), order=order)
    cfg = lmvd.make_config(w)
    print("plan memory", (w.n1, w.n2, w.n3), "order", order, flush=True)
    torch.cuda.synchronize()
    handles = [ctypes.c_void_p() for _ in range(4)]
    free = []  # from the first plan on: it brings the library's code and static memory along
    for h in handles:
        assert lmvd.library().lmvd_plan_create(ctypes.byref(cfg), ctypes.byref(h)) == 0
        free.append(torch.cuda.mem_get_info()[0])
    for h in handles:
        lmvd.library().lmvd_plan_destroy(h)
    once = 8.0 * 10 * (n2 + 1) * (w.n1 // 2) * (w.n3 // 2)
    print([a - b for a, b in zip(free, free[1:])], once, flush=True)
    assert (free[0] - free[-1]) / (len(handles) - 1) < 1.5 * once


def test_the_check_made_again_leaves_the_factors():
    """lmvd_factor_check with a limit of its own makes the factors again, whichever layout the plan has."""
    import torch
    from paper_2206_09878_amd.lmvd import Plan, Stepper
    w = workload("small", n=16, n2=33)
    a, b = (Stepper(Plan(w), make_inputs(w, seed=70, stage=0), stage=0) for _ in range(2))
    first = a.p.factor_check()
    assert a.p.factor_check(1e4) == first and first[3] == 0
    for s in (a, b):
        for _ in range(2):
            s.substep()
    for x, y in zip(state_tensors(a), state_tensors(b)):
        assert torch.equal(x, y)
