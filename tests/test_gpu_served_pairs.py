"""Served requests of a 16-bit stack whose pairs of plane elements are packed by the
requests themselves: every image, before and after, is bit for bit that of whole
records."""
import pytest

import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("store", ["f16", "bf16"])
def test_served_pairs(store):
    import torch
    import paper_2609_09322_amd as dart
    dims, M, P = (51, 43, 57), 6, 1024
    kind = {"f16": dart.DART_F16, "bf16": dart.DART_BF16}[store]
    j, b, times = synth.jet_torch(dims, M, 5, gamma_spine=4.0, n_knots=2)
    torch.cuda.synchronize()
    st = dart.dart_load_epochs(dims, (1, 1, 1), times, j, b, kind)
    records = dart.dart_stack_get_info(st).device_bytes
    L, tm = synth.diag(dims), 0.5 * (times[0] + times[-1])
    view = dart.View(40.0, 70.0, P, P, L / P, tm, 0.6)
    ref = torch.zeros((P, P), device="cuda")
    _, steps = dart.dart_render_batch([st], [dart.View(40.0, 70.0, P, P, L / P, tm, 0.6,
                                                       dart.DART_RECORDS_ONLY)], [ref])
    torch.cuda.synchronize()
    srv = dart.dart_server_create(256 << 20, 16, 2)
    try:
        for k in range(10):  # (80 requests of 79 million cells: the 51st makes 4e9)
            ims = [torch.full((P, P), -1.0, device="cuda") for _ in range(8)]
            torch.cuda.synchronize()
            tickets = [dart.dart_submit(srv, st, view, im) for im in ims]
            assert all(dart.dart_wait(srv, t)[1] == steps[0] for t in tickets)
            torch.cuda.synchronize()
            assert all(torch.equal(im, ref) for im in ims), k
            held = dart.dart_stack_get_info(st).device_bytes
            assert held == (records * 7 // 4 if k >= 7 else records * 5 // 4) or k == 6
    finally:
        dart.dart_server_destroy(srv)
