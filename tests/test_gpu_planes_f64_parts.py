"""Emissivity planes of FP64 stacks above 256 MiB as parts of labelled and vector stacks:
renders from the planes against whole-record renders (DART_RECORDS_ONLY), bit for bit,
plain and batched, with exact time (labelled) and after a part is refilled; and a
labelled stack one of whose parts is too small to have a plane."""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu

DIMS, M = (128, 128, 150), 4  # 315 MB of records


@pytest.mark.parametrize("kind", ["labelled", "vector", "labelled, one small"])
def test_planes_of_f64_parts(kind):
    import torch
    import paper_2609_09322_amd as dart
    j, b, times = synth.jet_torch(DIMS, M, 6, gamma_spine=4.0, n_knots=2)
    torch.cuda.synchronize()
    j, b = j.double(), b.double()
    j[1, 70:74] *= -1.0
    j[2, 80, 10:20] = -0.0
    parts, nz, depth = [], (DIMS[2], 20 if "small" in kind else DIMS[2]), 0
    for k in range(2):
        jj, bb = j[:, :nz[k]].contiguous(), b[:, :nz[k]].contiguous()
        p = dart.dart_load_epochs((DIMS[0], DIMS[1], nz[k]), (1, 1, 1), times,
                                  jj if k == 0 else 0.5 * jj, bb, dart.DART_F64)
        if kind != "vector":
            dart.dart_stack_set_placement(p, (0, 0, depth), (64, 64, 0.5 * sum(nz)))
            depth += nz[k]
        parts.append(p)
    st = (dart.dart_vector_create if kind == "vector" else dart.dart_labelled_create)(parts)
    P, L = 90, synth.diag((DIMS[0], DIMS[1], sum(nz)))
    shape = (2, P, P) if kind == "vector" else (P, P)
    stream = torch.cuda.Stream()

    def same(flags, plain=False):
        views = [dart.View(th, ph, P, P, L / P, 0.0, 0.6, flags | extra, dart.DART_F64)
                 for extra in (0, dart.DART_RECORDS_ONLY) for th, ph in ((25.0, 10.0), (80.0, 200.0))]
        im = [torch.full(shape, -1.0, dtype=torch.float64, device="cuda") for _ in views]
        if plain:
            steps = [dart.dart_render(st, v, x)[1] for v, x in zip(views, im)]
        else:
            steps = dart.dart_render_batch([st] * 4, views, im, stream=stream)[1]
        torch.cuda.synchronize()
        for k in range(2):
            a, c = im[k].cpu().numpy(), im[k + 2].cpu().numpy()
            assert np.array_equal(a.view(np.uint64), c.view(np.uint64)) and steps[k] == steps[k + 2]
            assert steps[k] > 0
        return im[0]

    for _ in range(3):  # (a labelled stack's planes come with its second render)
        first = same(0)
    same(dart.DART_NEAREST_EPOCH)
    same(dart.DART_PLANE_ADDR64)
    if kind != "vector":
        same(dart.DART_EXACT_TIME)
    same(0, plain=True)
    dart.dart_stack_set_epochs(parts[0], 1, (2.0 * j[1:3]).contiguous(), b[1:3].flip(1).contiguous())
    assert not torch.equal(same(0), first)
