"""A batch on a stream that its caller captures is refused: what is captured stays as
it is, and the batches after it are right."""
import pytest

import synth

pytestmark = pytest.mark.gpu


def _jet(dart, torch, store):
    dims, M = (48, 40, 60), 4
    j, b, times = synth.jet_torch(dims, M, 6, gamma_spine=4.0, n_knots=2)
    torch.cuda.synchronize()
    st = dart.dart_load_epochs(dims, (1, 1, 1), times, j, b, store)
    L = synth.diag(dims)
    return st, dart.View(40.0, 70.0, 100, 100, L / 100, 0.0, 0.6), j, b


def test_batch_under_capture_is_refused():
    import torch
    import paper_2609_09322_amd as dart
    st, view, _, _ = _jet(dart, torch, dart.DART_F32)
    ref = torch.zeros((100, 100), device="cuda")
    dart.dart_render(st, view, ref)
    im, x = torch.full((100, 100), -1.0, device="cuda"), torch.zeros(8, device="cuda")
    stream = torch.cuda.Stream()
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=stream, capture_error_mode="relaxed"):
        x += 1.0
        with pytest.raises(dart.DartError) as ei:
            dart.dart_render_batch([st], [view], [im], stream=stream, stats=False)
    assert ei.value.status == dart.DART_E_DEVICE
    for k in range(3):
        graph.replay()
        torch.cuda.synchronize()
        assert (x == k + 1.0).all() and (im == -1.0).all()
    for _ in range(3):
        im.fill_(-1.0)
        torch.cuda.synchronize()
        dart.dart_render_batch([st], [view], [im], stream=stream)
        assert torch.equal(im, ref)
