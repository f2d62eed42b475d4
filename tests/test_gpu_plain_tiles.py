"""The plain kernel's arrangements of an image (8 x 8 or 64 x 1 tiles with a ray's depth
segments side by side, rows of pixels with the segments in one lane), at image sides
around a tile, a workgroup and the rows that are dealt to the XCDs, and as strips of a
pixel or three: images bit for bit those of the batched kernel, cell-steps equal."""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu

# Cells a pixel: under 4 the tiles are square, or, for 257 to 1024 wavefronts of rays in
# whole records of these stacks (more than 384 MiB an epoch), rows of pixels; above 4,
# with fewer rays, 64 x 1.
IMAGES = [(1, 1), (8, 8), (1, 4099), (4097, 3), (65, 120), (129, 121), (63, 257), (300, 128), (40, 249),
          (251, 249), (701, 130)]
STACKS = {"f64": (230, 240, 235), "f32": (300, 290, 300), "f16": (376, 372, 370),
          "bf16": (376, 372, 370)}


@pytest.mark.parametrize("store", list(STACKS))
@pytest.mark.parametrize("vector", [False, True])
def test_arrangements(store, vector):
    import torch
    import paper_2609_09322_amd as dart
    kind = {"f64": dart.DART_F64, "f32": dart.DART_F32, "f16": dart.DART_F16,
            "bf16": dart.DART_BF16}[store]
    dims, M = STACKS[store], 2
    j, b, times = synth.jet_torch(dims, M, 5, gamma_spine=4.0, n_knots=2)
    torch.cuda.synchronize()
    if store == "f64":
        j, b = j.double(), b.double()
    st = parts = dart.dart_load_epochs(dims, (1, 1, 1), times, j, b, kind)
    if vector:
        parts = [st, dart.dart_load_epochs(dims, (1, 1, 1), times, 0.5 * j, b, kind)]
        st = dart.dart_vector_create(parts)
    del j, b
    out, td = ((dart.DART_F64, torch.float64) if store == "f64" else (dart.DART_F32, torch.float32))
    tm = 0.5 * (times[0] + times[-1])
    views = [dart.View(58.0 + 3 * k, 95.0 + k, W, H, ps, tm, 0.6, flags, out)
             for k, (W, H) in enumerate(IMAGES) for ps in (0.45, 2.0, 4.5)
             for flags in (0, dart.DART_RECORDS_ONLY)]
    shape = [((2, v.height, v.width) if vector else (v.height, v.width)) for v in views]
    batch = [torch.full(s, -1.0, dtype=td, device="cuda") for s in shape]
    _, steps = dart.dart_render_batch([st] * len(views), views, batch, stream=torch.cuda.Stream())
    torch.cuda.synchronize()
    for v, s, ref, n in zip(views, shape, batch, steps):
        im = torch.full(s, -2.0, dtype=td, device="cuda")
        _, m = dart.dart_render(st, v, im)
        assert m == n and torch.equal(im, ref), (v.width, v.height, v.pixel_scale, v.flags)
    assert sum(steps) > 0
