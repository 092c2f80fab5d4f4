"""Matrices whose lanes stand at a stated distance from each other, and which kernels that leaves them."""
import functools
import os
import subprocess
import tempfile

import numpy as np

import paper_2509_22951_amd as tq

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_2509_22951_amd", "csrc")


@functools.lru_cache(maxsize=None)
def _classifier():
    exe = os.path.join(tempfile.mkdtemp(prefix="tq_class_"), "driver")
    subprocess.run(["g++", "-std=c++17", "-O2", "-pthread", os.path.join(HERE, "ring_class_driver.cpp"), os.path.join(CSRC, "tq_blob.cpp"), "-o", exe], check=True)
    return exe


def _classify(blob):
    with tempfile.NamedTemporaryFile() as f:
        f.write(blob)
        f.flush()
        return [int(v) for v in subprocess.run([_classifier(), f.name], check=True, capture_output=True, text=True, timeout=60).stdout.split()]


def ring_class(blob):
    """2: k_matvec_ring and k_matvec_runs with rings of either size, 1: k_matvec_runs with rings of 128 bytes, 0: the whole-strip
    kernel (what the creation decides, by its own function)."""
    return _classify(blob)[0]


def lane_reach(blob):
    """Columns past the start of its segment that a lane reaches in the activation image of the dot-product kernel."""
    return _classify(blob)[1]


def _steps(rng, seg_cols, limit, spare):
    """Columns per chunk of 4 codes of the first row and of the others: the first takes pairs and the others single bytes until
    they are `limit` columns apart, then all take the same number, in bursts of pairs among others.  Without spare codes the others
    take pairs and the first row single bytes at the end, so that all need the same number of codes and none can wait."""
    steps, slow, gap, burst = [], 0, 0, 0
    closing = [] if spare else [(a, b) for b, a in _opening(limit)]
    end = seg_cols - sum(b for _, b in closing)
    for a, b in _opening(limit):
        steps.append((a, b))
        slow += b
    assert slow + 8 <= end
    while slow < end:
        burst = burst - 1 if burst else (6 if rng.integers(4) == 0 else 0)
        a = 8 if burst else int(rng.integers(4, 9))
        if not spare:               # whole chunks up to the closing ones
            left = end - slow
            a = left if left <= 8 else min(a, left - 4)
        steps.append((a, a))
        slow += a
    return steps + closing


def _opening(limit):
    return [(8, 4)] * (limit // 4) + [(4 + limit % 4, 4)] * (limit % 4 > 0)


def bytes_at_the_limit(seed, cols, seg_cols, limit, spare=True, rows=16):
    """Bands of bytes whose last units' lanes drift exactly `limit` columns apart when they are coded with the pairs (p, p + 32),
    p = 64..95, and single bytes (_steps, the same in all panels).  The units before hold single bytes alone.  -> bytes [rows, cols]"""
    rng = np.random.default_rng(seed)
    Q = rng.integers(1, 64, (rows, cols), dtype=np.uint8)
    steps = _steps(rng, seg_cols, limit, spare)
    unit = (cols - 1) // (4 * seg_cols) * (4 * seg_cols)
    for first in range(unit, cols, seg_cols):
        end = min(cols, first + seg_cols)
        for r in range(rows):
            at = first
            for step in steps:                  # a chunk: pairs for the columns beyond 4, then single bytes
                n = min(step[min(r % 16, 1)], end - at)
                for k in range(max(0, n - 4)):
                    Q[r, at + 2 * k] = rng.integers(64, 96)
                    Q[r, at + 2 * k + 1] = Q[r, at + 2 * k] + 32
                at += n
    return Q


def drifting(seed, cols, seg_cols, limit, opts, spare=True, rows=16):
    """bytes_at_the_limit as a container -> (weights, scales, container)."""
    Qb = bytes_at_the_limit(seed, cols, seg_cols, limit, spare, rows)
    pairs = np.array([[p, p + 32] for p in range(64, 96)], np.uint8).view(np.int8)
    d = tq.tq_encode_quantized(pairs, np.ones(32, np.float32), max_entries=288, dictionary="frequency")
    Q = Qb.view(np.int8)
    if opts:   # byte j of a row holds columns 2j and 2j + 1 as 4-bit values
        Q = np.stack([((Qb & 15) ^ 8).astype(np.int8) - 8, ((Qb >> 4) ^ 8).astype(np.int8) - 8], axis=2).reshape(Qb.shape[0], -1)
    scales = np.linspace(0.005, 0.015, Q.shape[0]).astype(np.float32)
    blob = tq.tq_encode_quantized(Q, scales, max_entries=288, seg_cols=seg_cols, dict_from=d, dictionary="frequency", **opts)
    assert tq.tq_validate_blob(blob)["lane_spread"] == limit
    return Q, scales, blob
