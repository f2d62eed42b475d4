"""Loads, re-lays and read-backs in blocks of whole bricks: grids at the edges of
the blocks (one cell, one row, one column, a cell more than a block, narrow and
ragged grids) under every kind of brick, every storage type.  The stored values
are the inputs (representable ones), so every pass must give them back exactly;
a bad value is reported at its own position wherever it lies in a block."""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu

DIMS = [(1, 1, 1), (65, 3, 5), (64, 16, 2), (1, 1, 700), (3, 300, 1), (257, 1, 2), (17, 33, 9)]
BRICKS = [(1, 1, 1), (16, 1, 1), (1, 16, 2), (1, 1, 16), (2, 4, 8), (16, 16, 16)]


@pytest.mark.parametrize("store", ["f64", "f32", "f16", "bf16"])
def test_blocks(store):
    import torch
    import paper_2609_09322_amd as dart
    kind = {"f64": dart.DART_F64, "f32": dart.DART_F32, "f16": dart.DART_F16,
            "bf16": dart.DART_BF16}[store]
    src = np.float64 if store == "f64" else np.float32
    held = {"f16": synth.round_f16, "bf16": synth.round_bf16}.get(store, lambda x: x)
    for k, dims in enumerate(DIMS):
        j, beta, times = synth.random_stack(dims, 3, seed=k, beta_max=0.9)
        j, beta = held(j.astype(src)), held(beta.astype(src))
        jd, bd = torch.from_numpy(j).cuda(), torch.from_numpy(beta).cuda()
        st = dart.dart_stack_create(dims, (1, 1, 1), times, kind)
        dart.dart_stack_set_epochs(st, 0, jd, bd)
        for brick in [None] + BRICKS:
            if brick is not None:
                dart.dart_stack_rebrick(st, brick)
                # (a refill under this brick shape)
                dart.dart_stack_set_epochs(st, 1, jd[1:].contiguous(), bd[1:].contiguous())
            for m in range(3):
                jr, br = np.empty_like(j[m]), np.empty_like(beta[m])
                dart.dart_stack_read_epoch(st, m, jr, br)
                assert np.array_equal(jr, j[m]) and np.array_equal(br, beta[m]), (dims, brick, m)
            # |beta| = 1 in one cell of epoch 1
            bad = bd[1:2].clone()
            z, y, x = (int(v) for v in np.unravel_index(
                (7 * j[0].size) // 9, j[0].shape))
            bad[0, z, y, x] = torch.tensor([0.0, 1.0, 0.0])
            with pytest.raises(dart.DartError) as ei:
                dart.dart_stack_set_epochs(st, 1, jd[1:2].contiguous(), bad)
            assert ei.value.status == dart.DART_E_RANGE
            assert f"epoch 1, cell (x={x}, y={y}, z={z})" in str(ei.value)
            dart.dart_stack_set_epochs(st, 1, jd[1:2].contiguous(), bd[1:2].contiguous())
