"""The emissivity plane of FP64 stacks (those above 256 MiB of records): renders
from the plane against whole-record renders of the same stack (DART_RECORDS_ONLY),
bit for bit, with the marks on moving, negative and -0 records, both address
forms, both ray marches, exact time, the plain kernel, and after a refill that keeps
the plane in step; and a smaller stack that stays without one."""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu


def test_plane_f64():
    import torch
    import paper_2609_09322_amd as dart
    dims, M = (128, 120, 140), 4  # 275 MB
    j, b, times = synth.jet_torch(dims, M, 3, gamma_spine=4.0, n_knots=3)
    torch.cuda.synchronize()
    j, b = j.double(), b.double()
    j[1, 60:64] *= -1.0
    j[2, 70, 10:20] = -0.0
    b[0, 30, 40:50, 5:9, 1] = -0.0
    st = dart.dart_load_epochs(dims, (1, 1, 1), times, j, b, dart.DART_F64)
    records = M * dims[0] * dims[1] * dims[2] * 32
    L = synth.diag(dims)
    stream = torch.cuda.Stream()

    def same(flags, plain=False):
        views = [dart.View(th, ph, 70, 70, L / 70, 0.0, 0.6, flags | extra, dart.DART_F64)
                 for extra in (0, dart.DART_RECORDS_ONLY) for th, ph in ((20.0, 10.0), (80.0, 200.0))]
        im = [torch.full((70, 70), -1.0, dtype=torch.float64, device="cuda") for _ in views]
        if plain:
            steps = [dart.dart_render(st, v, x)[1] for v, x in zip(views, im)]
        else:
            steps = dart.dart_render_batch([st] * 4, views, im, stream=stream)[1]
        torch.cuda.synchronize()
        for k in range(2):
            a, c = im[k].cpu().numpy(), im[k + 2].cpu().numpy()
            assert np.array_equal(a.view(np.uint64), c.view(np.uint64)) and steps[k] == steps[k + 2]
        return im[0]

    saved = dart.dart_get_tuning()
    try:
        for sync, cells in ((0, 4), (6, 8)):
            dart.dart_set_tuning(16, 4, 8, 0, 1, sync, cells)
            for flags in (0, dart.DART_EXACT_TIME, dart.DART_NEAREST_EPOCH, dart.DART_PLANE_ADDR64):
                first = same(flags)
        same(0, plain=True)
        assert dart.dart_stack_get_info(st).device_bytes == records + records // 4
        dart.dart_stack_set_epochs(st, 1, (2.0 * j[1:3]).contiguous(), b[1:3].flip(1).contiguous())
        assert not torch.equal(same(0), first)
    finally:
        dart.dart_set_tuning(saved.tile_w, saved.tile_h, saved.waves_per_cu, saved.order,
                             saved.orient, saved.depth_sync, saved.cells_per_batch or 4)
    small = dart.dart_load_epochs((32, 32, 32), (1, 1, 1), times[:2], j[:2, :32, :32, :32].contiguous(),
                                  b[:2, :32, :32, :32].contiguous(), dart.DART_F64)
    im = torch.zeros((40, 40), dtype=torch.float64, device="cuda")
    dart.dart_render(small, dart.View(30.0, 5.0, 40, 40, 1.5, 0.0, 0.6, 0, dart.DART_F64), im)
    assert dart.dart_stack_get_info(small).device_bytes == 2 * 32 ** 3 * 32
