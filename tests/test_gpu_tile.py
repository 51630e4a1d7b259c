"""Column kernels on LDS tiles (32, 16 or 8 columns per tile, the widest whose rows fit), GPU against the oracle:
row counts on both sides of every change of the tile width and of the streaming kernels' takeover, rows one
over and under a block of 16, column counts that leave the last tile ragged, and orders below the widest.
Tolerances: 1e-11, or the spread of the oracle's own results under other roundings where that is larger
(spread_tolerances)."""
import dataclasses

import pytest

from paper_2206_09878_amd.workloads import make_inputs, workload
from tests.test_gpu_parity import check_pair, gpu_substep, oracle_substep, spread_tolerances

pytestmark = pytest.mark.gpu


# tile width changes: m^c after 191 and 383 rows, prologue 127 and 287, right-hand sides 64, 144 and 256 (then
# streaming), projections 256
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
