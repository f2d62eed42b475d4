"""Nearest-epoch views of 16-bit stacks, in depth segments, against the FP64 oracle with
FP64 ray parameters: whether a midpoint halfway between two epochs goes to the one or the
other is decided as the oracle decides it, and the images agree to the precision of the
FP32 Doppler factors.  The tolerance: the hardware's log2 and exp2 are good to an ulp
and 1 + beta.s (at least 0.2 here) to 6e-8 absolute, which p = 2.6 times moves D^p by
less than 2e-6."""
import numpy as np
import pytest

import oracle
import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("store", ["f16", "bf16"])
@pytest.mark.parametrize("dims,side", [((64, 64, 64), 128), ((33, 47, 29), 64), ((120, 100, 140), 250)])
def test_nearest_epoch(store, dims, side):
    import paper_2609_09322_amd as dart
    L = float(np.sqrt(sum(n * n for n in dims)))
    times = np.linspace(-0.4 * L, 0.45 * L, 5)
    j, beta, _ = synth.random_stack(dims, 5, seed=7, beta_max=0.8, times=times, j_range=(0.1, 1.0))
    beta *= np.random.default_rng(7).random(j.shape)[..., None] < 0.1
    round_to = {"f16": synth.round_f16, "bf16": synth.round_bf16}[store]
    j, beta = round_to(j.astype(np.float32)), round_to(beta.astype(np.float32))
    kind = {"f16": dart.DART_F16, "bf16": dart.DART_BF16}[store]
    st = dart.dart_load_epochs(dims, (1, 1, 1), times, np.ascontiguousarray(j),
                               np.ascontiguousarray(beta), kind)
    ost = oracle.Stack(j.astype(np.float64), beta.astype(np.float64), times, cell=(1.0, 1.0, 1.0))
    for th, ph in ((37.0, 211.0), (71.0, 13.0)):
        view = dart.View(th, ph, side, side, 1.02 * L / side, 0.03, 0.6,
                         dart.DART_NEAREST_EPOCH | dart.DART_FORCE_F64_DDA)
        ref, steps = oracle.render(ost, oracle.View(th, ph, side, side, 1.02 * L / side, 0.03, 0.6,
                                                    dart.DART_NEAREST_EPOCH))
        plain, batch = (np.zeros((side, side), dtype=np.float32) for _ in range(2))
        _, n = dart.dart_render(st, view, plain)
        dart.dart_render_batch([st], [view], [batch])
        assert np.array_equal(plain, batch) and n == steps
        floor = 1e-3 * np.abs(ref).max()
        err = (np.abs(plain - ref) / np.maximum(np.abs(ref), floor)).max()
        assert err <= 2e-6, err
