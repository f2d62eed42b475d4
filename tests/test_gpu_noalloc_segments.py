"""The allocation-free batch where its scratch holds the sums of all its views' depth
segments, of some (the first views at once, the rest part after part on a wavefront) and
of none: images and cell-steps of the batched render, bit for bit, scalar and vector."""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("vector", [False, True])
@pytest.mark.parametrize("n,side", [(1, 1), (3, 65), (24, 300), (2000, 100)])
def test_scratch_for_segments(n, side, vector):
    import torch
    import paper_2609_09322_amd as dart
    # (a tile in 4 segments takes 2 KiB of sums: 24 x 1500 tiles of 300^2 pixels do not
    # fit 16 MiB whole; 2000 x 200 leave it little room)
    dims, M = (120, 100, 140), 4
    j, b, times = synth.jet_torch(dims, M, 5, gamma_spine=4.0, n_knots=2)
    torch.cuda.synchronize()
    st = dart.dart_load_epochs(dims, (1, 1, 1), times, j, b, dart.DART_F32)
    if vector:
        parts = [st, dart.dart_load_epochs(dims, (1, 1, 1), times, 0.5 * j, b, dart.DART_F32)]
        st = dart.dart_vector_create(parts)
    L = synth.diag(dims)
    views = [dart.View(20.0 + 0.07 * k, 0.17 * k, side, side, L / side, 0.0, 0.6,
                       (0, dart.DART_NEAREST_EPOCH, dart.DART_NO_LOOKBACK)[k % 3])
             for k in range(n)]
    shape = (2, side, side) if vector else (side, side)
    a = torch.full((n,) + shape, -1.0, device="cuda")
    c = torch.full_like(a, -2.0)
    stream = torch.cuda.Stream()
    torch.cuda.synchronize()
    _, na = dart.dart_render_batch([st] * n, views, list(a), stream=stream)
    _, nc = dart.dart_render_batch_noalloc([st] * n, views, list(c), stream=stream)
    torch.cuda.synchronize()
    assert torch.equal(a, c) and np.array_equal(na, nc)
    assert n == 1 or na.sum() > 0
