"""Depth segments: views of few, long rays are marched in 2 or 4 parts per ray.
Sizes at which a ray's parts can go wrong: grids and images around the rule's
edges, one-cell axes, axis-parallel and diagonal rays (ties of crossings at a
part's end), non-unit cells, windows that cut the rays, every storage type and
option.  Each image and its cell-steps against the FP64 oracle (the tolerances
of the parity tests, which are those of the storage types; cells belong to one
part each; counted on the oblique views, where no two crossings tie), and the batched kernel (a part per queue
item), the allocation-free one (part after part on one wavefront) and the plain
one (a part per wavefront of a workgroup) against each other, bit for bit."""
import numpy as np
import pytest

import oracle
import synth

pytestmark = pytest.mark.gpu

TOL = {"f64": 1e-12, "f32": 1e-5, "f16": 2e-3, "bf16": 2e-3}
# dims, cell, image sides
GRIDS = [((64, 64, 64), (1.0, 1.0, 1.0), (128, 128)),
         ((33, 47, 29), (1.0, 0.9, 1.2), (65, 63)),
         ((1, 70, 40), (2.0, 0.5, 0.75), (50, 31)),
         ((96, 2, 3), (0.5, 1.0, 1.0), (17, 90)),
         ((40, 40, 40), (1.0, 1.0, 1.0), (1, 1)),
         ((120, 100, 140), (1.0, 1.0, 1.0), (300, 280))]
ANGLES = [(90.0, 0.0), (0.0, 0.0), (90.0, 45.0), (37.0, 211.0), (54.735610317245346, 45.0)]


@pytest.mark.parametrize("store", ["f64", "f32", "f16", "bf16"])
@pytest.mark.parametrize("grid", range(len(GRIDS)))
def test_segments(store, grid):
    import torch
    import paper_2609_09322_amd as dart
    dims, cell, (W, H) = GRIDS[grid]
    nx, ny, nz = dims
    L = float(np.sqrt(sum((n * c) ** 2 for n, c in zip(dims, cell))))
    times = np.linspace(-0.4 * L, 0.45 * L, 5)  # the window ends inside the grid
    j, beta, _ = synth.random_stack(dims, 5, seed=40 + grid, beta_max=0.8, times=times,
                                    j_range=(0.1, 1.0))
    beta *= np.random.default_rng(grid).random(j.shape)[..., None] < 0.1  # mostly at rest
    src = np.float64 if store == "f64" else np.float32
    round_to = {"f16": synth.round_f16, "bf16": synth.round_bf16}.get(store, lambda x: x)
    j, beta = round_to(j.astype(src)), round_to(beta.astype(src))
    kind = {"f64": dart.DART_F64, "f32": dart.DART_F32, "f16": dart.DART_F16,
            "bf16": dart.DART_BF16}[store]
    st = dart.dart_load_epochs(dims, cell, times, np.ascontiguousarray(j),
                               np.ascontiguousarray(beta), kind)
    ost = oracle.Stack(j.astype(np.float64), beta.astype(np.float64), times, cell=cell)
    out = dart.DART_F64 if store == "f64" else dart.DART_F32
    views, refs = [], []
    for k, (th, ph) in enumerate(ANGLES):
        for flags in ((0, dart.DART_NEAREST_EPOCH, dart.DART_EXACT_TIME, dart.DART_NO_LOOKBACK,
                       dart.DART_FORCE_F64_DDA) if k == 3 else (0,)):
            views.append(dart.View(th, ph, W, H, 1.02 * L / max(W, H), 0.03, 0.6, flags, out))
            oflags = (flags & 7) | (oracle.EXACT_TIME if flags & dart.DART_EXACT_TIME else 0)
            refs.append(oracle.render(ost, oracle.View(th, ph, W, H, 1.02 * L / max(W, H), 0.03,
                                                       0.6, oflags)))
    t = torch.float64 if store == "f64" else torch.float32
    stream = torch.cuda.Stream()
    saved = dart.dart_get_tuning()
    try:
        for sync in (0, 6):
            dart.dart_set_tuning(16, 4, 8, 1 if sync else 4, 1, sync, 8)
            batch = [torch.full((H, W), -1.0, dtype=t, device="cuda") for _ in views]
            alone = [torch.full((H, W), -2.0, dtype=t, device="cuda") for _ in views]
            _, steps = dart.dart_render_batch([st] * len(views), views, batch, stream=stream)
            _, steps2 = dart.dart_render_batch_noalloc([st] * len(views), views, alone,
                                                       stream=stream)
            assert np.array_equal(steps, steps2)
            for k, v in enumerate(views):
                plain = np.zeros((H, W), dtype=src)
                _, n = dart.dart_render(st, v, plain)
                got = batch[k].cpu().numpy()
                assert np.array_equal(got, plain) and np.array_equal(alone[k].cpu().numpy(), plain)
                if store in ("f16", "bf16") and v.flags & dart.DART_NEAREST_EPOCH:
                    # (FP32 rays: a midpoint halfway between two epochs goes to
                    # either by rounding, and the other epoch's cell is another
                    # value; the whole-ray walk has the same pixel)
                    continue
                ref, ref_steps = refs[k]
                floor = 1e-3 * max(np.abs(ref).max(), 1e-300)
                err = (np.abs(got - ref) / np.maximum(np.abs(ref), floor)).max()
                assert err <= TOL[store], (dims, k, v.flags, err)
                assert n == steps[k]
                if ANGLES[min(3, k) if k < 8 else 4] == (37.0, 211.0):
                    # Crossings closer than their rounding swap: none in FP64
                    # rays; FP32 ones (16-bit stacks) round by 2^-24 of at most
                    # 100 cells, about 1e-5 of a cell per crossing.
                    loose = 1e-4 if store in ("f16", "bf16") else 0.0
                    assert abs(int(n) - ref_steps) <= 2 + loose * ref_steps
    finally:
        dart.dart_set_tuning(saved.tile_w, saved.tile_h, saved.waves_per_cu, saved.order,
                             saved.orient, saved.depth_sync, saved.cells_per_batch or 4)
