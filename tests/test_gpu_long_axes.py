"""FP32 rays count an axis's crossings up to 2048, the most cells an axis may
have with them; grids with a longer axis take FP64 rays.  Grids at that edge,
one long axis each, viewed along it from both ends, along the others and
obliquely, in the batched, the allocation-free and the plain kernel, against the
FP64 oracle.

Tolerance: a crossing of FP32 rays is off by the roundings of its plane and of
its base, at most 1.5 * 2^-24 of the extent L; a pixel by that at both ends of
its chord times j <= 1 (matter at rest), twice over for the shares that
neighbouring cells exchange, and by the storage type's relative 2e-3."""
import numpy as np
import pytest

import oracle
import synth

pytestmark = pytest.mark.gpu

ANGLES = [(90.0, 0.0), (90.0, 180.0), (90.0, 90.0), (90.0, 270.0), (0.0, 0.0), (180.0, 0.0),
          (83.0, 4.0), (41.0, 214.0)]


@pytest.mark.parametrize("n", [2047, 2048, 2049])
@pytest.mark.parametrize("axis", [0, 1, 2])
def test_long_axis(axis, n):
    import torch
    import paper_2609_09322_amd as dart
    dims = [5, 3, 4]
    dims[axis] = n
    L = float(np.sqrt(sum(d * d for d in dims)))
    times = np.linspace(-0.45 * L, 0.4 * L, 3)  # the window ends inside a long view's chords
    j, beta, _ = synth.random_stack(tuple(dims), 3, seed=n + axis, beta_max=0.0, times=times,
                                    j_range=(0.1, 1.0))
    j = synth.round_f16(j.astype(np.float32))
    beta = np.zeros_like(beta, dtype=np.float32)
    st = dart.dart_load_epochs(tuple(dims), (1.0, 1.0, 1.0), times, np.ascontiguousarray(j), beta,
                               dart.DART_F16)
    ost = oracle.Stack(j.astype(np.float64), beta.astype(np.float64), times)
    W, H = 21, 18
    views, forced = [], []
    for th, ph in ANGLES:
        views.append(dart.View(th, ph, W, H, 8.0 / W, 0.0, 0.6, 0, dart.DART_F32))
        forced.append(dart.View(th, ph, W, H, 8.0 / W, 0.0, 0.6, dart.DART_FORCE_F64_DDA,
                                dart.DART_F32))
    stream = torch.cuda.Stream()
    images = lambda: [torch.full((H, W), -1.0, device="cuda") for _ in views]
    batch, alone, in64 = images(), images(), images()
    _, steps = dart.dart_render_batch([st] * len(views), views, batch, stream=stream)
    _, steps2 = dart.dart_render_batch_noalloc([st] * len(views), views, alone, stream=stream)
    dart.dart_render_batch([st] * len(views), forced, in64, stream=stream)
    assert np.array_equal(steps, steps2)
    for k, v in enumerate(views):
        got = batch[k].cpu().numpy()
        plain = np.zeros((H, W), dtype=np.float32)
        _, count = dart.dart_render(st, v, plain)
        assert count == steps[k]
        assert np.array_equal(got, plain) and np.array_equal(alone[k].cpu().numpy(), plain)
        if n > 2048:
            assert np.array_equal(got, in64[k].cpu().numpy())
        ref, ref_steps = oracle.render(ost, oracle.View(*ANGLES[k], W, H, v.pixel_scale, 0.0, 0.6,
                                                        0))
        tol = 2e-3 * np.abs(ref) + 2 * 2 * 1.5 * 2.0 ** -24 * L
        assert (np.abs(got - ref) <= tol).all(), (dims, k, np.abs(got - ref).max())
        assert count > 0 and np.abs(ref).max() > 0
