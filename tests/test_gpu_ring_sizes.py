"""The batched kernels around the distance between lanes up to which rings of 64 bytes do, and the runs kernel with such rings."""
import numpy as np
import pytest
import torch

import paper_2509_22951_amd as tq
from drifting import drifting, ring_class
from inputs import make_activations, make_weights, small_case
from oracle import oracle as O
from test_gpu_work_split import TOL, _gated, _stream

pytestmark = pytest.mark.gpu


SHAPES = [(2048, 256, {}), (384, 96, {}), (1024, 128, {"pack": True})]
LANES = [(32, True, 2), (33, True, 2), (34, True, 2), (40, True, 2), (32, False, 2), (33, False, 2), (34, False, 1), (40, False, 1)]


# (lanes without a code to spare need room for the codes that close the distance again)
@pytest.mark.parametrize("cols,seg_cols,opts,limit,spare,kind", [s + l for s in SHAPES for l in LANES if l[1] or s[1] >= 3 * l[0] + 8])
def test_lanes_around_the_limit_of_the_small_ring(cols, seg_cols, opts, limit, spare, kind):
    """Lanes that can wait are brought within 33 columns when the matrix is loaded, whatever they were, and take the ring kernel; so do
    lanes that cannot but are no further apart; beyond that the runs kernel takes the matrix, with rings of 128 bytes."""
    Q, scales, blob = drifting(1, cols, seg_cols, limit, opts, spare)
    assert ring_class(blob) == kind
    m = tq.Matrix(blob)
    tq.tq_set_ring_min_bands_per_cu(0)
    try:
        for batch in (3, 8, 16):
            bits, x = make_activations(small_case(16, Q.shape[1], seed=batch), batch)
            ref = O.gemv_f64(Q, scales, x)
            gated, most = _gated(ref)
            xd = torch.from_numpy(bits.view(np.int16).copy()).cuda()
            y = torch.full((batch, 16), float("nan"), dtype=torch.float32, device="cuda")
            g = torch.full((batch, 8), float("nan"), dtype=torch.float32, device="cuda")
            m.matvec(xd.data_ptr(), y.data_ptr(), batch, _stream())
            tq.tq_matvec_gate_up(m.handle, xd.data_ptr(), g.data_ptr(), batch, _stream())
            torch.cuda.synchronize()
            for got, want, limits in ((y, ref, TOL * np.abs(ref).max(axis=1, keepdims=True)), (g, gated, most)):
                got = got.cpu().numpy().astype(np.float64)
                assert np.isfinite(got).all() and (np.abs(got - want) <= limits).all()
    finally:
        tq.tq_set_ring_min_bands_per_cu(24)
        m.close()


@pytest.mark.parametrize("rows,cols,seg_cols", [
    (16, 256, 256),       # one unit of one panel for one workgroup, cut into runs
    (250, 1000, 256),     # one ragged unit a band, rows past the end
    (700, 1999, 256),     # two units a band, odd rows of x, a last panel that ends inside a piece
    (4112, 1040, 128),    # more bands than workgroups: whole units, three a band, the last one a panel of 16 columns
    (4099, 2056, 512),    # segments of 512 columns, 257 bands
])
def test_small_shares_at_the_batches_that_take_the_small_rings(rows, cols, seg_cols):
    spec = small_case(rows, cols, seed=rows + cols)
    W = make_weights(spec)
    Q, scales = O.quantize_rows(W)
    m = tq.Matrix(tq.tq_encode(W, seg_cols=seg_cols))
    try:
        for batch, shift in ((4, 0), (5, 0), (8, 1), (9, 0), (16, 1)):
            bits, x = make_activations(spec, batch)
            ref = O.gemv_f64(Q, scales, x)
            xd = torch.from_numpy(np.concatenate([np.zeros(shift, np.int16), bits.view(np.int16).reshape(-1)])).cuda()[shift:]
            y = torch.full((batch, rows), float("nan"), dtype=torch.float32, device="cuda")
            m.matvec(xd.data_ptr(), y.data_ptr(), batch, _stream())
            torch.cuda.synchronize()
            got = y.cpu().numpy().astype(np.float64)
            assert np.isfinite(got).all() and (np.abs(got - ref).max(axis=1) <= TOL * np.abs(ref).max(axis=1)).all()
    finally:
        m.close()


def test_callers_own_line_between_the_batched_kernels():
    """tq_set_ring_min_bands_per_cu: bands per compute unit from which on a launch goes to the ring kernel, half as many above 8 rows
    of x; a matrix that only the runs kernel takes shows by a launch of its own.  Both ways give the product."""
    n_cu = torch.cuda.get_device_properties(0).multi_processor_count
    rows = 16 * (2 * n_cu + 1)
    specs = [small_case(rows, 256, seed=1), small_case(40, 300, seed=2)]
    Ws = [make_weights(s) for s in specs]
    refs = [O.quantize_rows(W) for W in Ws]
    mats = [tq.Matrix(tq.tq_encode(W, seg_cols=64, max_entries=600)) for W in Ws]
    try:
        for line, batch, launches in ((0, 3, 2), (1, 3, 2), (2, 8, 2), (3, 8, 1), (3, 9, 2), (5, 16, 2), (6, 16, 1), (1 << 31, 16, 1)):
            xs, ys, want = [], [], []
            for s, (Q, scales) in zip(specs, refs):
                bits, x = make_activations(s, batch)
                xs.append(torch.from_numpy(bits.view(np.int16).copy()).cuda())
                ys.append(torch.full((batch, s.rows), float("nan"), dtype=torch.float32, device="cuda"))
                want.append(O.gemv_f64(Q, scales, x))
            tq.tq_set_ring_min_bands_per_cu(line)
            step = tq.Step([m.handle for m in mats], [x.data_ptr() for x in xs], [y.data_ptr() for y in ys], batch)
            assert step.info["n_launches"] == launches, (line, batch)
            step.launch(_stream())
            torch.cuda.synchronize()
            step.close()
            for y, ref in zip(ys, want):
                got = y.cpu().numpy().astype(np.float64)
                assert np.isfinite(got).all() and (np.abs(got - ref).max(axis=1) <= TOL * np.abs(ref).max(axis=1)).all()
    finally:
        tq.tq_set_ring_min_bands_per_cu(24)
        for m in mats:
            m.close()
