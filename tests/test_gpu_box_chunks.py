"""The data-derived root box at the edges of its chunks (2048 particles, or n / 1024
of large sets; four particles a thread and step): every extreme is put on a single
particle at the edge, and the box must be exactly that of the data."""
import math

import numpy as np
import pytest
import torch

from paper_2312_06102_amd import treebuild as tb

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [6, 255, 1025, 2047, 2048, 2049, 4097, 2 ** 21 + 1, 2 ** 21 + 1025])
def test_extremes_at_chunk_edges(n):
    rng = np.random.default_rng(n)
    pos = rng.uniform(-1.0, 1.0, (n, 3)).astype(np.float32)
    edges = sorted({0, n - 1, min(n - 1, 2047), min(n - 1, 2048), n // 2, n - 2})
    for k, i in enumerate(edges):
        pos[i] = (3.0 + k, -2.0 - k, (-1.0) ** k * (4.0 + k))
    mass = np.full(n, 1.0 / n, np.float32)
    b = tb.Builder(n, 16)
    b.launch(torch.from_numpy(pos).cuda(), torch.from_numpy(mass).cuda())
    box = b.result()["box"].cpu().numpy()
    lo = pos.astype(np.float64).min(0)
    ext = float((pos.astype(np.float64).max(0) - lo).max())
    assert np.array_equal(box[:3], lo)
    assert box[3] == math.ldexp(1.0, math.frexp(ext)[1])
