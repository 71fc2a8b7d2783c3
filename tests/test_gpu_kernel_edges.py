"""Edges of kernels and of the rules that pick them, against the CPU oracle: sizes around tiles, remainders and
the smallest and largest of a kernel's range."""
import numpy as np
import pytest

import oracle
from skl_harness import build_states_on_gpu

pytestmark = pytest.mark.gpu


def hash_params(rng, d):
    return (2 * rng.integers(0, 1 << 23, size=d) + 1).astype(np.uint32), rng.integers(0, 1 << 24, size=d).astype(np.uint32)


@pytest.mark.parametrize("in_f,out_f,d,widths", [
    (2051, 264, 4, (8, 33)),         # eight channels per workgroup, the last one with three; whole 16-byte pieces
    (2048, 333, 3, (10,)),           # rows not aligned to 16 bytes
    (70, 1030, 2, (16, 64)),         # few channels: one per workgroup
    (515, 96, 8, (250, 3)),          # tables that leave room for fewer channels per workgroup
    (3, 65536, 2, (500,)),           # the most outputs a 32-bit key can number
    (3, 65544, 2, (500,)),           # one step beyond: 64-bit keys
])
def test_row_sketch_construction(in_f, out_f, d, widths):
    """Bit-identical to the oracle's sequential update (integers: no tolerance)."""
    rng = np.random.default_rng(in_f + out_f)
    W = (rng.standard_normal((in_f, out_f)) * 0.02).astype(np.float16)
    W[:, ::3] = np.float16(0.0078125) * rng.choice(np.array([-1, 1], dtype=np.float16), size=W[:, ::3].shape)     # ties of both signs
    K = np.array([widths[j % len(widths)] for j in range(in_f)], dtype=np.uint32)
    A, C = hash_params(rng, d)
    got = build_states_on_gpu(W, 1, out_f, d, A, C, K)
    assert np.array_equal(got, oracle.update(W, 1, out_f, d, A, C, K).states)
