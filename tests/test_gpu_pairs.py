"""Pairs of plane elements (a record's and the next epoch's in one word), which
batches of a 16-bit stack read once its records have been walked enough.  Every image is compared
bit for bit with the same batch's from whole records: odd grids, bricks that leave an epoch a whole or an odd number of
words of four, windows that end at the last epoch, options that read the plane
instead (one epoch per cell, exact time, 64-bit addresses), marked records
(moving, negative, -0), a refill and a re-lay."""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu

# dims, epochs, bricks (the last FP16 one: more than 4 GiB of pairs, two windows)
CASES = {"f16": [((151, 143, 157), 10, None), ((51, 43, 57), 11, (1, 1, 1)),
                 ((384, 380, 384), 21, (1, 2, 8))],
         "bf16": [((64, 257, 230), 9, (1, 2, 16)), ((17, 299, 333), 2, (2, 1, 1))]}


@pytest.mark.parametrize("store,case", [(s, c) for s in CASES for c in range(len(CASES[s]))])
def test_pairs_equal_records(store, case):
    import torch
    import paper_2609_09322_amd as dart
    dims, M, brick = CASES[store][case]
    kind = {"f16": dart.DART_F16, "bf16": dart.DART_BF16}[store]
    j, b, times = synth.jet_torch(dims, M, 5, gamma_spine=4.0, n_knots=2)
    flat = j.view(-1)
    flat[1::1013] *= -1.0
    flat[7::4001] = -0.0
    st = dart.dart_load_epochs(dims, (1.0, 1.0, 1.0), times, j, b, kind)
    if brick:
        dart.dart_stack_rebrick(st, brick)
    L = float(np.sqrt(sum(d * d for d in dims)))
    W = 70
    views, marks = [], (0, 0, dart.DART_NEAREST_EPOCH, dart.DART_EXACT_TIME, dart.DART_NO_LOOKBACK,
                        dart.DART_FORCE_F64_DDA, dart.DART_PLANE_ADDR64)
    tm = 0.5 * (times[0] + times[-1])
    for k, f in enumerate(marks):
        views.append(dart.View(31.0 + 17.0 * k, 200.0 + 31.0 * k, W, W - k, L / W,
                               tm + (0.2 * L if k == 1 else 0.0), 0.6, f, dart.DART_F32))
    whole = [dart.View(v.theta_deg, v.phi_deg, v.width, v.height, v.pixel_scale, v.t_obs, v.alpha,
                       v.flags | dart.DART_RECORDS_ONLY, v.out_dtype) for v in views]
    stream = torch.cuda.Stream()
    saved = dart.dart_get_tuning()

    def images():
        return [torch.full((v.height, v.width), -1.0, device="cuda") for v in views]

    def batch(vs, call=dart.dart_render_batch):
        im = images()
        _, steps = call([st] * len(vs), vs, im, stream=stream)
        return [i.cpu().numpy().view(np.uint32) for i in im], steps

    big = [dart.View(40.0, 70.0, 1024, 1024, L / 1024, tm, 0.6, 0, dart.DART_F32)]
    bigs = torch.zeros((1024, 1024), device="cuda")

    def walk():
        # 4e9 cells and 16 per record, at half the sum of the axes for each ray
        need = (4e9 + 16 * records // 8) / (0.5 * sum(dims) * 1024 ** 2)
        for _ in range(int(need) + 1):
            dart.dart_render_batch([st], big, [bigs], stream=stream, stats=False)

    def same():
        for sync, cells in ((0, 4), (6, 8)):
            dart.dart_set_tuning(16, 4, 8, 0, 1, sync, cells)
            ref, n = batch(whole)
            assert n.sum() > 0
            for call in (dart.dart_render_batch, dart.dart_render_batch_noalloc):
                got, m = batch(views, call)
                assert np.array_equal(n, m)
                for k in range(len(views)):
                    assert np.array_equal(got[k], ref[k]), (sync, cells, k)

    def held():
        return dart.dart_stack_get_info(st).device_bytes

    try:
        batch(views)
        records = held() * 4 // 5  # the records and a plane of a quarter of them
        assert held() == records + records // 4
        walk()
        assert held() == records + records // 4 + records // 2
        same()
        # a refill: the plane until its records have been walked, then pairs again
        m = M // 2
        dart.dart_stack_set_epochs(st, m, (1.5 * j[m:m + 1]).contiguous(),
                                   b[m:m + 1].flip(1).contiguous())
        same()
        walk()
        same()
        dart.dart_stack_rebrick(st, (2, 4, 4))
        same()
        records = held() * 4 // 5
        walk()
        assert held() == records + records // 4 + records // 2
        same()
    finally:
        dart.dart_set_tuning(saved.tile_w, saved.tile_h, saved.waves_per_cu, saved.order,
                             saved.orient, saved.depth_sync, saved.cells_per_batch or 4)
        dart.dart_free_epochs(st)
