"""How a launch's work is cut: units shared between the wavefronts of a workgroup, whole workgroups per matrix.  Small shapes at
the edges of the rules, every output against the float64 product."""
import numpy as np
import pytest
import torch

import paper_2509_22951_amd as tq
from inputs import make_activations, make_weights, small_case
from oracle import oracle as O

pytestmark = pytest.mark.gpu

# Sums of exact products in fp32 over at most K terms: the error is below K * 2^-24 of the sum of magnitudes in the worst
# case and about its square root in practice; 1e-5 of the largest output is far above either's typical size here
# (K <= 4096, measured 2e-7) and far below what one misplaced column would show (1e-2).
TOL = 1e-5


def _stream():
    return torch.cuda.current_stream().cuda_stream


class _Job:
    def __init__(self, rows, cols, batch, seed, **opts):
        spec = small_case(rows, cols, seed=seed)
        W = make_weights(spec)
        self.Q, s = O.quantize_rows(W, opts.get("bits", 8))
        bits, x = make_activations(spec, batch)
        self.ref = O.gemv_f64(self.Q, s, x)
        self.m = tq.Matrix(tq.tq_encode(W, **opts))
        self.x = torch.from_numpy(bits.view(np.int16).copy()).cuda()
        self.y = torch.full((batch, rows), float("nan"), dtype=torch.float32, device="cuda")

    def check(self):
        y = self.y.cpu().numpy().astype(np.float64)
        for got, ref in zip(y, self.ref):
            assert np.isfinite(got).all() and np.abs(got - ref).max() <= TOL * np.abs(ref).max()


SHARES = [
    # rows, cols, seg_cols: units of a workgroup's share (whole bands of quads) and their length
    (16, 8, 16),          # one unit of two chunks for 8 or 12 wavefronts: most runs are empty
    (16, 250, 64),        # one unit
    (16, 3000, 64),       # one band of 12 units, the last one part empty
    (16, 4096, 32),       # one band of 32 units: as many as are never shared
    (16, 3968, 32),       # 31 units: still shared between 8 wavefronts
    (4099, 1500, 128),    # one or two bands of 3 units, ragged rows and columns
    (8192, 512, 32),      # two bands of 4 units: a whole unit each for 8 wavefronts
]


@pytest.mark.parametrize("opts", [{}, {"bits": 4, "pack": True}], ids=["bytes", "packed"])
@pytest.mark.parametrize("batch", [1, 2])
@pytest.mark.parametrize("rows,cols,seg_cols", SHARES)
def test_units_shared_between_wavefronts(rows, cols, seg_cols, batch, opts):
    job = _Job(rows, cols, batch, seed=rows + cols, seg_cols=seg_cols, **opts)
    try:
        job.m.matvec(job.x.data_ptr(), job.y.data_ptr(), batch, _stream())
        torch.cuda.synchronize()
        job.check()
    finally:
        job.m.close()


@pytest.mark.parametrize("n", [2, 7, 32, 33])   # 32: the most matrices that get whole workgroups
def test_matrices_of_a_call_get_whole_workgroups(n):
    jobs = [_Job(16 * (1 + (37 * i) % 60) + i % 3, 256 * (1 + i % 4) + i % 2, 1, seed=100 + i, seg_cols=64, max_entries=600) for i in range(n)]
    try:
        call = tq.MultiCall([j.m.handle for j in jobs], [j.x.data_ptr() for j in jobs], [j.y.data_ptr() for j in jobs], 1)
        call.launch(_stream())
        torch.cuda.synchronize()
        for j in jobs:
            j.check()
            j.y.fill_(float("nan"))
        stages = [i // 5 for i in range(n)]      # the same as a staged step, launched again and again
        step = tq.Step([j.m.handle for j in jobs], [j.x.data_ptr() for j in jobs], [j.y.data_ptr() for j in jobs], 1, stages=stages)
        assert step.info["persistent"] == 1
        for _ in range(3):
            step.launch(_stream())
            torch.cuda.synchronize()
            for j in jobs:
                j.check()
                j.y.fill_(float("nan"))
        step.close()
    finally:
        for j in jobs:
            j.m.close()
