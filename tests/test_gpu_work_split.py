"""How a launch's work is cut: units shared between the wavefronts of a workgroup, whole workgroups per matrix.  Small shapes at
the edges of the rules, every output against the float64 product."""
import numpy as np
import pytest
import torch

import paper_2509_22951_amd as tq
from drifting import drifting, ring_class
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
        self.x_of = lambda shift: torch.from_numpy(np.concatenate([np.zeros(shift, np.int16), bits.view(np.int16).reshape(-1)])).cuda()[shift:]
        self.x = torch.from_numpy(bits.view(np.int16).copy()).cuda()
        self.y = torch.full((batch, rows), float("nan"), dtype=torch.float32, device="cuda")

    def check(self):
        y = self.y.cpu().numpy().astype(np.float64)
        for got, ref in zip(y, self.ref):
            assert np.isfinite(got).all() and np.abs(got - ref).max() <= TOL * np.abs(ref).max()


SHARES = [
    # rows, cols, seg_cols: units of a workgroup's share (whole bands of quads) and their length.  Units are shared between 8 wavefronts
    # in shares of 1 to 6, 9 to 12, 17 and 18, between 12 (packed) in shares of up to 6.
    (16, 8, 16),          # one unit of two chunks for 8 or 12 wavefronts: most runs are empty
    (16, 250, 64),        # one unit
    (16, 500, 64),        # two units (packed: one)
    (16, 700, 64),        # three units (packed: two)
    (16, 1500, 64),       # six units, the most of the first kind (packed: three)
    (16, 2000, 64),       # eight units: a whole one each (packed: four)
    (16, 3000, 64),       # one band of 12 units, the last one part empty (packed: six)
    (16, 4096, 32),       # one band of 32 units
    (16, 3968, 32),       # 31 units: one wavefront has one less
    (4099, 1500, 128),    # one or two bands of 3 units, ragged rows and columns
    (8192, 512, 32),      # two bands of 4 units: a whole unit each for 8 wavefronts
    (16, 4600, 64),       # 18 units, two to a wavefront and two over
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


# Runs that start inside a unit, at any chunk of it: at marks and between them, marks of two bytes (segments over 510 columns),
# shares of one to one and a half units to a wavefront.
STARTS = [
    (16, 4096, 1024),     # one unit of 128 chunks or more, 16 marks
    (37, 3000, 1008),     # three bands, the last one and the last panel ragged
    (16, 1900, 496),      # the widest segments with marks of a byte
    (16, 9 * 256, 64),    # nine units of 8 or 9 chunks: one mark or none
    (16, 11 * 1024 - 3, 256),
    (9000, 257, 512),     # one panel; two or three bands to a workgroup
]


@pytest.mark.parametrize("opts", [{}, {"bits": 4, "pack": True}], ids=["bytes", "packed"])
@pytest.mark.parametrize("batch", [1, 2, 3, 7, 16])
@pytest.mark.parametrize("rows,cols,seg_cols", STARTS)
def test_runs_that_start_inside_a_unit(rows, cols, seg_cols, batch, opts):
    if opts and cols % 2:
        cols += 1
    job = _Job(rows, cols, batch, seed=rows + cols + batch, seg_cols=seg_cols, **opts)
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


# Stages whose workgroups take equal numbers of units: bands of 2, 3, 4 and 8 quads that two workgroups share, ragged last bands,
# matrices beside each other.  (The first stage has a band for every workgroup, as clearing ahead needs it.  Which stages share is
# plan_driver.cpp's to say; packed matrices never do, nor outputs in one place.)
SHARED = [
    [[(4096, 256)], [(2033, 2048)], [(5111, 768)], [(3000, 768), (1000, 768)]],       # shares of 4 of 8, 4 of 3; 3 of 3: whole bands
    [[(4096, 256)], [(2048, 512), (3072, 512)], [(3072, 2000)], [(2048, 1000)]],      # 3 of 2, 6 of 8, 2 of 4
]


@pytest.mark.parametrize("opts", [{}, {"bits": 4, "pack": True}], ids=["bytes", "packed"])
@pytest.mark.parametrize("batch", [1, 2])
@pytest.mark.parametrize("one_place", [False, True], ids=["own outputs", "outputs in one place"])
@pytest.mark.parametrize("shapes", SHARED)
def test_bands_that_workgroups_of_a_stage_share(shapes, one_place, batch, opts):
    jobs = [[_Job(r, c, batch, seed=7 * k + r + c, seg_cols=32 if opts else 64, **opts) for r, c in stage] for k, stage in enumerate(shapes)]
    flat = [j for stage in jobs for j in stage]
    stages = [k for k, stage in enumerate(jobs) for _ in stage]
    try:
        if one_place:     # a stage's outputs over those of the stage before: they must not be cleared while that one is in work
            place = torch.empty(max(sum(j.y.numel() for j in stage) for stage in jobs), dtype=torch.float32, device="cuda")
            for stage in jobs:
                at = 0
                for j in stage:
                    j.y = place[at:at + j.y.numel()].view_as(j.y)
                    at += j.y.numel()
        step = tq.Step([j.m.handle for j in flat], [j.x.data_ptr() for j in flat], [j.y.data_ptr() for j in flat], batch, stages=stages)
        assert step.info["persistent"] == 1
        before = None
        for _ in range(4):
            for j in flat:
                j.y.fill_(float("nan"))
            step.launch(_stream())
            torch.cuda.synchronize()
            checked = jobs[-1] if one_place else flat
            for j in checked:
                j.check()
            got = [j.y.clone() for j in checked]
            assert before is None or all(torch.equal(a, b) for a, b in zip(before, got))     # the sums do not depend on timing
            before = got
        step.close()
    finally:
        for j in flat:
            j.m.close()


class _Exact:
    """Stages of 2048 x 2048 in segments of 64, four units of every band's eight for each of two workgroups, with activations at one column
    of a segment and 3 powers of two between the quads: what a wavefront sums is exact, and what is rounded are the band's sums alone."""
    SHAPES = [(4096, 256), (2048, 2048), (2048, 2048), (2048, 2048)]     # (plan_driver.cpp: stages 1, 2, 3 share)

    def __init__(self, batch=1):
        rng = np.random.default_rng(7)
        self.batch, self.mats, self.xs, self.scale, self.total = batch, [], [], [], []
        for rows, cols in self.SHAPES:
            q = rng.integers(-127, 128, (rows, cols), dtype=np.int8)
            scale = rng.uniform(0.5, 1.0, rows).astype(np.float32)
            quads = np.array([0, 2, 4, 6, 1, 3, 5, 7])[: cols // 256]
            x = np.zeros((batch, cols // 256, 4, 64), np.float32)
            x[..., 9] = rng.integers(128, 256, x.shape[:3]) * rng.choice([-1, 1], x.shape[:3]) * 2.0 ** (-3 * quads)[:, None]
            x = x.reshape(batch, cols)
            self.total.append(x.astype(np.float64) @ q.T.astype(np.float64))
            self.scale.append(scale)
            self.mats.append(tq.Matrix(tq.tq_encode_quantized(q, scale, seg_cols=64)))
            self.xs.append(torch.from_numpy(x).cuda().to(torch.bfloat16))

    def run(self, ys):
        step = tq.Step([m.handle for m in self.mats], [x.data_ptr() for x in self.xs], [y.data_ptr() for y in ys], self.batch, stages=list(range(len(self.mats))))
        assert step.info["persistent"] == 1
        step.launch(_stream())
        torch.cuda.synchronize()
        step.close()
        return [y.cpu().numpy() for y in ys]

    def whole(self, k):      # a band's sum in double, rounded once, times its scale
        return self.total[k].astype(np.float32) * self.scale[k]

    def error(self, k, y):
        exact = self.total[k] * self.scale[k].astype(np.float64)
        return np.linalg.norm(y - exact) / np.linalg.norm(exact)


@pytest.mark.parametrize("batch", [1, 2])
def test_bands_that_workgroups_share_are_rounded_no_further_than_whole_ones(batch):
    """Two parts, each rounded once, and their sum, against a sum that is rounded before and after its scale: the same error (here 3.56e-8
    for 3.56e-8; with the parts rounded before and after their scale 4.29e-8).  Where outputs cannot be added to the bands are whole: then
    every bit is that of the sum in double."""
    e = _Exact(batch)
    try:
        fresh = lambda **kw: [torch.full((batch, r), float("nan"), dtype=torch.float32, **kw) for r, _ in e.SHAPES]
        got = e.run(fresh(device="cuda"))
        assert np.array_equal(got[0], e.whole(0))
        for k in (1, 2, 3):
            assert not np.array_equal(got[k], e.whole(k))     # (two workgroups have been at it)
        shared, whole = (np.mean([e.error(k, y[k]) for k in (1, 2, 3)]) for y in (got, [e.whole(k) for k in range(4)]))
        assert shared <= 1.05 * whole, (shared, whole)        # (18432 roundings of one spread: 1 % of it)
        host = e.run(fresh(pin_memory=True))
        place = torch.full((batch, 4096), float("nan"), dtype=torch.float32, device="cuda").view(-1)
        over = e.run([place[:batch * r].view(batch, r) for r, _ in e.SHAPES])
        for k in (1, 2, 3):
            assert np.array_equal(host[k], e.whole(k))
        assert np.array_equal(over[3], e.whole(3))
    finally:
        for m in e.mats:
            m.close()


def _chain():
    """A stage whose activations are the shared outputs of the stage before: small whole numbers as fp32 are pairs (0, the number) of bf16."""
    rng = np.random.default_rng(3)
    shapes = [(4096, 256), (2048, 2048), (2048, 4096)]       # (plan_driver.cpp: stages 1 and 2 share)
    q = [rng.integers(-1, 2, s, dtype=np.int8) for s in shapes]
    q[2][:, rng.permutation(4096)[:3800]] = 0                # (148 or so of its columns meet a number: sums below 2^24)
    x0, x1 = (np.where(np.arange(c) % 32 == 5, rng.integers(-1, 2, c), 0).astype(np.float32) for c in (256, 2048))
    y1 = q[1].astype(np.int64) @ x1.astype(np.int64)
    pairs = np.zeros(4096, np.int64)
    pairs[1::2] = y1
    assert np.abs(y1).max() < 256
    refs = [q[0].astype(np.int64) @ x0.astype(np.int64), y1, q[2].astype(np.int64) @ pairs]
    mats = [tq.Matrix(tq.tq_encode_quantized(w, np.ones(len(w), np.float32), seg_cols=64)) for w in q]
    ys = [torch.full((r,), float("nan"), dtype=torch.float32, device="cuda") for r, _ in shapes]
    xs = [torch.from_numpy(x0).cuda().to(torch.bfloat16), torch.from_numpy(x1).cuda().to(torch.bfloat16), ys[1]]
    step = tq.Step([m.handle for m in mats], [x.data_ptr() for x in xs], [y.data_ptr() for y in ys], 1, stages=[0, 1, 2])
    return mats, xs, ys, refs, step


@pytest.mark.parametrize("replayed", [False, True], ids=["launched", "in a graph"])
def test_a_stage_reads_what_two_workgroups_added_to_in_the_stage_before(replayed):
    mats, xs, ys, refs, step = _chain()
    try:
        assert step.info["persistent"] == 1
        graph = None
        if replayed:
            graph = torch.cuda.CUDAGraph()
            with torch.cuda.graph(graph, stream=torch.cuda.Stream()):
                step.launch(torch.cuda.current_stream().cuda_stream)
        for turn in range(6):
            for y in ys:
                y.fill_(float("nan"))
            torch.cuda.synchronize()
            if replayed and turn % 3 != 2:
                graph.replay()
            else:
                step.launch(_stream())          # (eager work between the replays)
            torch.cuda.synchronize()
            for y, ref in zip(ys, refs):
                assert np.array_equal(y.cpu().numpy(), ref.astype(np.float32))
        assert tq.tq_step_get_info(step.handle)["fault"] == 0
        del graph
    finally:
        step.close()
        for m in mats:
            m.close()


# More bands than compute units, fewer than 8 stored columns: whole workgroups per matrix at the narrow end.
NARROW = [(6, {}), (3, {}), (1, {}), (10, {"bits": 4, "pack": True}), (14, {"bits": 4, "pack": True})]


@pytest.mark.parametrize("cols,opts", NARROW)
@pytest.mark.parametrize("rows", [4800, 4099 * 3])
def test_narrow_matrices_with_more_bands_than_workgroups(rows, cols, opts):
    for batch in (1, 2, 3):       # the dot-product kernel, the runs kernel (or, narrower than a fragment, the whole-strip kernel)
        job = _Job(rows, cols, batch, seed=rows + cols, seg_cols=16, **opts)
        try:
            job.m.matvec(job.x.data_ptr(), job.y.data_ptr(), batch, _stream())
            torch.cuda.synchronize()
            job.check()
            if batch == 1:
                job.y.fill_(float("nan"))
                step = tq.Step([job.m.handle], [job.x.data_ptr()], [job.y.data_ptr()], 1, stages=[0])
                assert step.info["persistent"] == 1
                step.launch(_stream())
                torch.cuda.synchronize()
                step.close()
                job.check()
        finally:
            job.m.close()


RUNS = [
    # rows, cols, seg_cols: batches above 2 below the sizes the ring kernel with an activation tile takes
    (16, 6, 16),           # narrower than an activation fragment: the whole-strip kernel
    (16, 8, 16),           # one fragment
    (17, 42, 64),          # a segment that ends inside an 8-byte piece of the ring
    (33, 300, 48),         # segments of one and a half groups of windows, the last one short
    (40, 1021, 256),       # one unit per band, row ends inside a fragment
    (100, 4095, 1024),     # the widest segments
    (5000, 2999, 256),     # bands shared between wavefronts, a dictionary's start (units that are levelled)
]


@pytest.mark.parametrize("opts", [{}, {"bits": 4, "pack": True}], ids=["bytes", "packed"])
@pytest.mark.parametrize("batch,shift", [(3, 0), (8, 1), (16, 0)])
@pytest.mark.parametrize("rows,cols,seg_cols", RUNS)
def test_runs_of_units_in_batches(rows, cols, seg_cols, batch, shift, opts):
    job = _Job(rows, cols + cols % 2 if opts else cols, batch, seed=rows + cols, seg_cols=seg_cols, **opts)
    try:
        x = job.x_of(shift)       # rows of x at odd addresses
        job.m.matvec(x.data_ptr(), job.y.data_ptr(), batch, _stream())
        torch.cuda.synchronize()
        job.check()
    finally:
        job.m.close()


@pytest.mark.parametrize("opts", [{}, {"pack": True}], ids=["bytes", "packed"])
@pytest.mark.parametrize("cols,seg_cols,limit,spare,kind", [
    # Seven units for one workgroup, taken whole: the last one ends inside a piece of the ring.  (With this seed the first row stands
    # a whole ring past what has been multiplied at 1 look per panel of 128 bytes, 5 of 64.)  Lanes that can wait are brought
    # together when the matrix is loaded; those that cannot stand as far apart as the rings of 64 and of 128 bytes take.
    (7 * 4 * 1008 - 12, 1008, 65, True, 2),
    (7 * 4 * 1008 - 12, 1008, 113, True, 2),
    (7 * 4 * 1008 - 12, 1008, 33, False, 2),
    (7 * 4 * 1008 - 12, 1008, 34, False, 1),
    (7 * 4 * 1008 - 12, 1008, 65, False, 1),
    # one unit, cut between the wavefronts
    (500, 512, 65, True, 2),
    (500, 512, 113, True, 2),
    (500, 512, 33, False, 2),
    (500, 512, 66, False, 1),      # (the rows end ahead of the last chunk: a few codes to spare)
])
def test_lanes_as_far_apart_as_the_rings_take(cols, seg_cols, limit, spare, kind, opts):
    """k_matvec_runs with rings of 128 bytes (kind 1) and of either size (kind 2)."""
    Q, scales, blob = drifting(2, cols, seg_cols, limit, opts, spare)
    assert ring_class(blob) == kind
    m = tq.Matrix(blob)
    try:
        for batch in (3, 8, 16):
            bits, x = make_activations(small_case(16, Q.shape[1], seed=batch), batch)
            ref = O.gemv_f64(Q, scales, x)
            xd = torch.from_numpy(bits.view(np.int16).copy()).cuda()
            y = torch.full((batch, Q.shape[0]), float("nan"), dtype=torch.float32, device="cuda")
            for _ in range(2):
                m.matvec(xd.data_ptr(), y.data_ptr(), batch, _stream())
            torch.cuda.synchronize()
            for got, want in zip(y.cpu().numpy().astype(np.float64), ref):
                assert np.isfinite(got).all() and np.abs(got - want).max() <= TOL * np.abs(want).max()
    finally:
        m.close()


def _gated(ref):
    """silu(gate) * up of the even and odd rows of a product, and how far it may be off: both sums are within e = TOL * max |ref| of a
    batch row; |silu'| <= 1.1 and |silu(g)| <= |g|, so the gated product is within e * (1.1 |up| + |gate|) (and e^2)."""
    gate, up = ref[:, 0::2], ref[:, 1::2]
    e = TOL * np.abs(ref).max(axis=1, keepdims=True)
    return gate / (1.0 + np.exp(-gate)) * up, e * (1.1 * np.abs(up) + np.abs(gate) + e)


@pytest.mark.parametrize("opts", [{}, {"pack": True}], ids=["bytes", "packed"])
@pytest.mark.parametrize("cols,seg_cols,limit", [(2048, 512, 66), (2048, 512, 114), (4096, 512, 150), (500, 512, 150)])
def test_lanes_further_apart_than_the_rings_take(cols, seg_cols, limit, opts):
    """The whole-strip kernel: whole units and a ragged one, 16-byte aligned x and x at odd addresses, products and gated pairs."""
    Q, scales, blob = drifting(3, cols, seg_cols, limit, opts, spare=False)
    assert ring_class(blob) == 0
    m = tq.Matrix(blob)
    try:
        for batch, shift in ((3, 0), (5, 1), (16, 0)):
            bits, x = make_activations(small_case(16, Q.shape[1], seed=batch), batch)
            ref = O.gemv_f64(Q, scales, x)
            gated, most = _gated(ref)
            xd = torch.from_numpy(np.concatenate([np.zeros(shift, np.int16), bits.view(np.int16).reshape(-1)])).cuda()[shift:]
            y = torch.full((batch, 16), float("nan"), dtype=torch.float32, device="cuda")
            g = torch.full((batch, 8), float("nan"), dtype=torch.float32, device="cuda")
            m.matvec(xd.data_ptr(), y.data_ptr(), batch, _stream())
            tq.tq_matvec_gate_up(m.handle, xd.data_ptr(), g.data_ptr(), batch, _stream())
            torch.cuda.synchronize()
            for got, want, limits in ((y, ref, TOL * np.abs(ref).max(axis=1, keepdims=True)), (g, gated, most)):
                got = got.cpu().numpy().astype(np.float64)
                assert np.isfinite(got).all() and (np.abs(got - want) <= limits).all()
    finally:
        m.close()


@pytest.mark.parametrize("opts", [{}, {"pack": True}], ids=["bytes", "packed"])
@pytest.mark.parametrize("gate_up", [False, True])
def test_matrices_for_all_three_batched_kernels_in_one_call(gate_up, opts):
    """Lanes 33, 65 and 80 columns apart that cannot wait, several bands each: a launch of the ring kernel, one of the runs kernel
    (which takes the second matrix, and the first too where the first's x is at an odd address) and one of the whole-strip kernel."""
    most = (1024, 128) if opts else (2048, 256)      # the widest segments of the ring kernel
    mats = [drifting(20 + i, *(most if limit == 33 else (2048, 256)), limit, opts, spare=False, rows=rows)
            for i, (limit, rows) in enumerate([(33, 96), (65, 80), (80, 48), (33, 16), (34, 4112)])]
    assert [ring_class(blob) for _, _, blob in mats] == [2, 1, 0, 2, 1]
    hs = [tq.Matrix(blob) for _, _, blob in mats]
    tq.tq_set_ring_min_bands_per_cu(0)
    try:
        for batch in (3, 8, 16):
            for shift in (0, 1):
                xs, ys, refs = [], [], []
                for i, (Q, scales, _) in enumerate(mats):
                    bits, x = make_activations(small_case(16, Q.shape[1], seed=10 * batch + i), batch)
                    odd = shift if i in (0, 3) else 0
                    xs.append(torch.from_numpy(np.concatenate([np.zeros(odd, np.int16), bits.view(np.int16).reshape(-1)])).cuda()[odd:])
                    refs.append(O.gemv_f64(Q, scales, x))
                    ys.append(torch.full((batch, Q.shape[0] // (2 if gate_up else 1)), float("nan"), dtype=torch.float32, device="cuda"))
                args = [h.handle for h in hs], [x.data_ptr() for x in xs], [y.data_ptr() for y in ys], batch
                step = tq.Step(*args, gate_up=gate_up)
                assert step.info["n_launches"] == (2 if shift else 3)
                for through_step in (True, False):
                    for y in ys:
                        y.fill_(float("nan"))
                    if through_step:
                        step.launch(_stream())
                    elif gate_up:
                        tq.tq_matvec_gate_up_multi(*args, _stream())
                    else:
                        tq.tq_matvec_multi(*args, _stream())
                    torch.cuda.synchronize()
                    for y, ref in zip(ys, refs):
                        want, most = _gated(ref) if gate_up else (ref, TOL * np.abs(ref).max(axis=1, keepdims=True))
                        got = y.cpu().numpy().astype(np.float64)
                        assert np.isfinite(got).all() and (np.abs(got - want) <= most).all()
                step.close()
    finally:
        tq.tq_set_ring_min_bands_per_cu(24)
        for h in hs:
            h.close()


@pytest.mark.parametrize("opts", [{}, {"bits": 4, "pack": True}], ids=["bytes", "packed"])
@pytest.mark.parametrize("batch", [3, 16])
@pytest.mark.parametrize("rows", [72, 33 * 256 * 8])      # gate rows: one band per workgroup; a pass of 32 bands and one more
def test_gated_pairs_on_the_ring_kernel(rows, batch, opts):
    cols = 512 if opts else 256
    spec = small_case(rows, cols, seed=5)
    Wg, Wu = make_weights(spec), make_weights(small_case(rows, cols, seed=6))
    bits, x = make_activations(spec, batch)
    width = opts.get("bits", 8)
    ref = O.gate_up_f64(*O.quantize_rows(Wg, width), *O.quantize_rows(Wu, width), x)
    m = tq.Matrix(tq.tq_encode_gate_up(Wg, Wu, seg_cols=32, **opts))
    xd = torch.from_numpy(bits.view(np.int16).copy()).cuda()
    y = torch.full((batch, rows), float("nan"), dtype=torch.float32, device="cuda")
    tq.tq_set_ring_min_bands_per_cu(0)
    try:
        tq.tq_matvec_gate_up(m.handle, xd.data_ptr(), y.data_ptr(), batch, _stream())
        torch.cuda.synchronize()
    finally:
        tq.tq_set_ring_min_bands_per_cu(24)
        m.close()
    y = y.cpu().numpy().astype(np.float64)
    for got, want in zip(y, ref):      # silu adds the rounding of exp and a division in fp32, relative to each output
        assert np.isfinite(got).all() and np.abs(got - want).max() <= 2 * TOL * np.abs(want).max()


@pytest.mark.parametrize("shift", [0, 4, 1])              # 16-, 4- and 1-byte stores
@pytest.mark.parametrize("escapes", [0, 3])
@pytest.mark.parametrize("marker,raw", [(2047, 1), (2047, 2), (2047, 3), (2046, 2), (2046, 3), (2045, 3), (2044, 3), (4095, 3)])
def test_listing_streams_whose_last_block_starts_no_token(marker, raw, escapes, shift):
    """Streams of 2048-word blocks that end in a marker at word `marker` with `raw` values, which lie in a block of their own
    (one block earlier for (2044, 3): the block ends with them).  Bytes around the output stay as they are."""
    table = np.full((1, 4), 7, np.uint8)
    values = np.concatenate([np.arange(4 * escapes, dtype=np.uint8), np.full(4 * (marker - 5 * escapes), 7, np.uint8),
                             np.arange(raw, dtype=np.uint8)])
    words = tq.tq_listing_compress(values, table)
    assert words[marker] == 0xFFFF and words.size == marker + 1 + raw
    h = tq.Listing(words, table)
    guard = 64
    buf = torch.full((guard + shift + values.size + guard,), 99, dtype=torch.uint8, device="cuda")
    try:
        h.decompress(buf[guard + shift:].data_ptr(), _stream())
        torch.cuda.synchronize()
    finally:
        h.close()
    got = buf.cpu().numpy()
    assert np.array_equal(got[guard + shift:guard + shift + values.size], values)
    assert (got[:guard + shift] == 99).all() and (got[guard + shift + values.size:] == 99).all()


def test_replayed_staged_step_waits_again_after_one_that_gave_up():
    """A staged step whose last product reads what the one before it wrote (an fp32 output of small whole numbers is, read as
    bf16, zeros and those numbers in turn), behind stages that keep one workgroup busy for longer than the others
    would poll in a launch that has given up.  Captured, launched once with no polls allowed, replayed: the replay waits."""
    rng = np.random.default_rng(4)
    jobs = [_Job(16, 16384, 1, seed=40 + i, seg_cols=256, max_entries=600) for i in range(4)]
    Qb = rng.integers(-1, 2, (16, 512)).astype(np.int8)
    xb = np.where(np.arange(512) < 100, np.uint16(0x3F80), np.uint16(0))      # bf16 1.0 a hundred times
    Qc = rng.integers(-100, 101, (4096, 32)).astype(np.int8)
    b = tq.Matrix(tq.tq_encode_quantized(Qb, np.ones(16, np.float32), max_entries=600))
    c = tq.Matrix(tq.tq_encode_quantized(Qc, np.ones(4096, np.float32), max_entries=600))
    yb_ref = Qb[:, :100].astype(np.int64).sum(axis=1)
    yc_ref = Qc[:, 1::2].astype(np.int64) @ yb_ref
    xbd = torch.from_numpy(xb.view(np.int16)).cuda()
    yb = torch.zeros(16, dtype=torch.float32, device="cuda")
    yc = torch.zeros(4096, dtype=torch.float32, device="cuda")
    busy = [jobs[i % 4] for i in range(60)]
    step = tq.Step([j.m.handle for j in busy] + [b.handle, c.handle], [j.x.data_ptr() for j in busy] + [xbd.data_ptr(), yb.data_ptr()],
                   [j.y.data_ptr() for j in busy] + [yb.data_ptr(), yc.data_ptr()], 1, stages=list(range(62)))
    try:
        assert step.info["persistent"] == 1
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=torch.cuda.Stream()):
            step.launch(_stream())
        for gave_up in (False, True, True):
            if gave_up:
                tq.tq_step_set_spin_limit(step.handle, 0)
                if tq.tq_step_get_info(step.handle)["fault"] == 0:
                    step.launch(_stream())
                torch.cuda.synchronize()
                assert tq.tq_step_get_info(step.handle)["fault"] == 1
            yb.zero_()
            yc.fill_(float("nan"))
            torch.cuda.synchronize()
            graph.replay()
            torch.cuda.synchronize()
            assert np.array_equal(yb.cpu().numpy(), yb_ref) and np.array_equal(yc.cpu().numpy(), yc_ref)
        del graph
    finally:
        step.close()
        for m in [j.m for j in jobs] + [b, c]:
            m.close()
