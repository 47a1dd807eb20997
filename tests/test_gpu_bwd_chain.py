"""The fused chain of input gradients (head, shared FFN, output projection) at the
edges of its window tiles: batches of one window, past a 16-window tile, and past
the line where tiles widen to 32; FFN widths of one chunk and several; weights
per repeat; every model width."""
import numpy as np
import pytest

import oracle as O
import synth
from gpu_helpers import to_dev

pytestmark = pytest.mark.gpu

TINY = dict(W=16, e=16, g=4, H=1, F=256, k=2)
CASES = [("fp32", TINY, 4100, False), ("bf16", TINY, 4100, False), ("bf16", TINY, 1, False),
         ("bf16", dict(W=32, e=32, g=4, H=4, F=512, k=2), 17, False),
         ("bf16", dict(W=32, e=32, g=8, H=8, F=768, k=3), 33, True),
         ("fp32", dict(W=32, e=32, g=8, H=8, F=512, k=2), 18, True),
         ("bf16", dict(W=32, e=64, g=8, H=8, F=512, k=2), 19, False)]


@pytest.mark.parametrize("dtype,shape,n,untied", CASES)
def test_gradients_match_oracle(dtype, shape, n, untied):
    import paper_2203_16114_amd as P
    cfg = O.Config(**shape, untied=untied)
    W = shape["W"]
    streams = synth.random_streams(31, n, W + 3)
    flat = synth.random_flat(6, O.init_flat(cfg, 1).size, 0.05)
    m = P.TraceModel(**shape, dtype=dtype, untied_ffn=untied, max_windows=n, max_keep=n)
    m.init_weights(0, 0.02, flat)
    m.forward_bits(to_dev(streams), W + 1, 1, keep=True)
    m.adapt_step()
    got = O.unflatten(m.grads(), cfg)
    w, y = O.windows_at(streams, np.arange(n), np.full(n, W + 1), W)
    _, ref = O.forward_backward(flat, cfg, w, y, mode="fp64" if dtype == "fp32" else "bf16")
    for k, r in ref.items():
        if dtype == "fp32":
            assert np.all(np.abs(got[k] - r) <= 1e-4 * np.abs(r) + 1e-5 * np.abs(r).max()), k
        else:  # the same bf16 storage points, sums in another order: 1e-2 by norm
            assert np.linalg.norm(got[k] - r) <= 1e-2 * np.linalg.norm(r), k
