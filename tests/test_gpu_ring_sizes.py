"""The ring kernel with rings of 64 and of 128 bytes, around the distance between lanes where one takes over from the other."""
import numpy as np
import pytest
import torch

import paper_2509_22951_amd as tq
from inputs import make_activations, make_weights, small_case
from oracle import oracle as O
from test_gpu_work_split import TOL, _drifting, _stream

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("cols,seg_cols,opts", [(2048, 256, {}), (384, 96, {}), (1024, 128, {"pack": True})], ids=["256", "96", "packed"])
@pytest.mark.parametrize("limit", [32, 33, 34, 40])
def test_lanes_around_the_limit_of_the_small_ring(cols, seg_cols, opts, limit):
    Q, scales, m = _drifting(5, cols, seg_cols, limit, opts)
    tq.tq_set_ring_min_bands_per_cu(0)
    try:
        for batch in (3, 8, 16):
            bits, x = make_activations(small_case(16, Q.shape[1], seed=batch), batch)
            ref = O.gemv_f64(Q, scales, x)
            gate, up = ref[:, 0::2], ref[:, 1::2]
            gated = gate / (1.0 + np.exp(-gate)) * up
            # Both sums are within e = TOL * max |ref| of a batch row; |silu'| <= 1.1 and |silu(g)| <= |g|, so the gated product is
            # within e * (1.1 |up| + |gate|) (and e^2).  (Relative to the row's largest output it may be far off: where every
            # gate of a batch row is well below zero, silu(g) ~ g exp(g) turns an error of the sum into a factor.)
            e = TOL * np.abs(ref).max(axis=1, keepdims=True)
            limits = (e, e * (1.1 * np.abs(up) + np.abs(gate) + e))
            xd = torch.from_numpy(bits.view(np.int16).copy()).cuda()
            y = torch.full((batch, 16), float("nan"), dtype=torch.float32, device="cuda")
            g = torch.full((batch, 8), float("nan"), dtype=torch.float32, device="cuda")
            m.matvec(xd.data_ptr(), y.data_ptr(), batch, _stream())
            tq.tq_matvec_gate_up(m.handle, xd.data_ptr(), g.data_ptr(), batch, _stream())
            torch.cuda.synchronize()
            for got, want, most in ((y, ref, limits[0]), (g, gated, limits[1])):
                got = got.cpu().numpy().astype(np.float64)
                assert np.isfinite(got).all() and (np.abs(got - want) <= most).all()
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
