"""Two served requests with one device destination, in waves that run at the same
time: a long dense render, and one that is done at once (no epoch is seen, every
pixel 0).  Whichever ends last, the image is one of the two from corner to corner,
and a third request to it, sent while both are in flight, changes nothing about that."""
import time

import pytest

import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("third", [False, True])
def test_one_destination_two_waves(third):
    import torch
    import paper_2609_09322_amd as dart
    dims, M, P = (256, 256, 256), 8, 4096
    j, b, times = synth.jet_torch(dims, M, 5, gamma_spine=4.0, n_knots=2)
    torch.cuda.synchronize()
    st = dart.dart_load_epochs(dims, (1, 1, 1), times, j + 1.0, b, dart.DART_F16)
    del j, b
    L, tm = synth.diag(dims), 0.5 * (times[0] + times[-1])
    dense = dart.View(40.0, 70.0, P, P, L / P, tm, 0.6, dart.DART_FORCE_F64_DDA)
    empty = dart.View(40.0, 70.0, P, P, L / P, tm + 1e6, 0.6)
    ref = torch.zeros((P, P), device="cuda")
    dart.dart_render_batch([st], [dense], [ref], stream=torch.cuda.Stream())
    torch.cuda.synchronize()
    assert (ref > 0).float().mean() > 0.3
    saved = dart.dart_get_tuning()
    dart.dart_set_tuning(32, 2, 4, 0, 1, 0, 4)  # (one wave per SIMD: room for another wave's)
    srv = dart.dart_server_create(3 << 30, 16, 3)
    try:
        for k in range(4):
            im = torch.full((P, P), -1.0, device="cuda")
            torch.cuda.synchronize()
            waves = dart.dart_server_get_stats(srv).waves
            tickets = [dart.dart_submit(srv, st, dense, im)]
            while dart.dart_server_get_stats(srv).waves == waves:
                time.sleep(1e-5)
            tickets.append(dart.dart_submit(srv, st, empty, im))
            if third:
                tickets.append(dart.dart_submit(srv, st, dense, im))
            done = [dart.dart_wait(srv, t) for t in tickets]
            print([f"{d[2]:.2f} ms" for d in done], flush=True)
            assert done[0][1] > 10 ** 9 and done[1][1] == 0
            torch.cuda.synchronize()
            wrong = min(int((im != ref).sum()), int((im != 0).sum()))
            assert wrong == 0, (k, wrong)
    finally:
        dart.dart_server_destroy(srv)
        dart.dart_set_tuning(saved.tile_w, saved.tile_h, saved.waves_per_cu, saved.order,
                             saved.orient, saved.depth_sync, saved.cells_per_batch or 4)
