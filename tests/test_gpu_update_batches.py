"""The update's batch-size rules: weight gradients grouped into one launch or not,
the embedding gradient from slices of the window bytes (up to 2^20 positions) or
from the counting sort."""
import numpy as np
import pytest

import oracle as O
import synth
from gpu_helpers import make_model, ocfg, to_dev, workload_cfg

pytestmark = pytest.mark.gpu


def _grads(m, s, W, cfg):
    m.forward_bits(s, W, 1, keep=True)
    m.adapt_step()
    return O.unflatten(m.grads(), cfg)


@pytest.mark.parametrize("wid,dtype", [(1, "fp32"), (4, "bf16")])
def test_repeated_batch_keeps_its_gradient(wid, dtype):
    """The gradient is a mean over windows: a batch repeated 8 or 17 times, past
    every batch-size rule (17 x 4100 windows of 16 or 32 bytes are more than 2^20
    positions), has the gradient of one copy within the sums' rounding."""
    shape, _ = workload_cfg(wid)
    cfg = ocfg(**shape)
    W, n = shape["W"], 4100
    s = to_dev(synth.random_streams(41, n, W + 1))
    flat = synth.random_flat(8, O.init_flat(cfg, 1).size, 0.05)
    one = _grads(make_model(shape, dtype, 0, max_windows=n, max_keep=n, flat=flat), s, W, cfg)
    for r in (8, 17):
        m = make_model(shape, dtype, 0, max_windows=r * n, max_keep=r * n, flat=flat)
        many = _grads(m, s.repeat(r, 1), W, cfg)
        for k, g in one.items():
            # fp32 sums of 4100 r terms; bf16: dz / (r n) rounds anew at a storage point (2^-9)
            tol = 1e-5 if dtype == "fp32" else 5e-3
            assert np.linalg.norm(many[k] - g) <= tol * np.linalg.norm(g), (r, k)


@pytest.mark.parametrize("n", [1, 511, 513, 1025])
def test_embedding_slices(n):
    """One slice of 16384 positions, its edge, and two and three: skewed bytes and
    one single byte, against the oracle."""
    shape, _ = workload_cfg(2)
    cfg = ocfg(**shape)
    W = shape["W"]
    rng = np.random.default_rng(n)
    for streams in (rng.choice([7, 7, 7, 7, 32, 255], size=(n, W + 1)).astype(np.uint8),
                    np.full((n, W + 1), 65, np.uint8)):
        flat = synth.random_flat(9, O.init_flat(cfg, 1).size, 0.05)
        m = make_model(shape, "fp32", 0, max_windows=n, max_keep=n, flat=flat)
        got = _grads(m, to_dev(streams), W, cfg)["E"]
        w, y = O.windows_at(streams, np.arange(n), np.full(n, W), W)
        _, ref = O.forward_backward(flat, cfg, w, y, mode="fp64")
        r = ref["E"]
        assert np.all(np.abs(got - r) <= 1e-4 * np.abs(r) + 1e-5 * np.abs(r).max())
        assert not np.any(got[1:7]) and not np.any(got[100:200])  # bytes that do not occur
