"""The coder's per-position kernel (frequencies, interval of the byte, decoded
byte in one pass) against the general path: trace_quantize of each position's
logits and the host range coder on the frequency rows, byte for byte."""
import numpy as np
import pytest

import paper_2203_16114_amd as P
from gpu_helpers import to_dev

pytestmark = pytest.mark.gpu

SHAPE = dict(W=16, e=16, g=4, H=1, F=256, k=2, dtype="fp32")


# one stream, partial and whole workgroups (4 streams each), one host thread
# (below 4096 streams) and several
@pytest.mark.parametrize("B", [1, 3, 4, 5, 257, 4099])
def test_codes_are_the_general_paths(B):
    import torch
    W, n = SHAPE["W"], 3
    rng = np.random.default_rng(B)
    flat = (0.3 * rng.standard_normal(P.param_count(P.make_config(**SHAPE)))).astype(np.float32)
    streams = rng.integers(0, 256, (B, W + n), dtype=np.uint8)
    streams[:, W] = np.arange(B) % 256  # every byte value, the first and the last of a lane among them
    streams[:, W + 1] = 255 - np.arange(B) % 256
    models = []
    for _ in range(2):
        m = P.TraceModel(**SHAPE, max_windows=B)
        m.init_weights(0, flat=flat)
        models.append(m)
    s = to_dev(streams)
    freq = np.ones((B, W + n, 256), np.uint16)  # the first W bytes at 1/256
    for i in range(W, W + n):
        z = models[0].forward_bits(s, i, 1, logits=True)["logits"]
        f = P.quantize(z)
        torch.cuda.synchronize()
        freq[:, i] = f.cpu().numpy().view(np.uint16)
    codes, _ = models[0].compress(s)
    for b in range(B):
        assert codes[b] == P.rc_encode(freq[b], streams[b]), b
    back, _ = models[1].decompress(codes, W + n)
    assert np.array_equal(back.cpu().numpy(), streams)
