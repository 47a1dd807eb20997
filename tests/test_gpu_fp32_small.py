"""The fp32 kernels of small launches: the FFN and head on 16- and 32-window
tiles, and the update's products whose k range is split over a workgroup's
waves.  Window counts sit at the edges of the tiles and of the dispatch."""
import numpy as np
import pytest
import torch

import oracle as O
import synth
from gpu_helpers import check_parity, make_model, ocfg, to_dev, workload_cfg

pytestmark = pytest.mark.gpu

D256 = dict(W=32, e=32, g=8, H=8, F=512, k=2)


def _shape(which):
    return D256 if which == "d256" else workload_cfg(which)[0]


@pytest.mark.parametrize("which,edge", [(1, 32768), (2, 32768), ("d256", 16384)])
def test_ffn_tiles_give_the_same_bits(which, edge):
    """A window's logits and code length do not depend on the launch: 16-window
    tiles (up to 4096 windows), 32-window tiles (below 256 wide tiles) and the
    wide tiles (from `edge` windows on) agree bit for bit; a sample agrees with
    the oracle."""
    shape = _shape(which)
    W = shape["W"]
    streams = synth.random_streams(7, edge, W + 1)
    s = to_dev(streams)
    m = make_model(shape, "fp32", 11, max_windows=edge)
    ref = m.forward_bits(s, W, 1, logits=True)
    z, b = ref["logits"].clone(), ref["bits"].clone()
    for n in (1, 15, 17, 4096, 4097, edge - 1):
        r = m.forward_bits(s[:n].contiguous(), W, 1, logits=True)
        assert torch.equal(r["logits"].view(torch.int32), z[:n].view(torch.int32)), n
        assert torch.equal(r["bits"].view(torch.int32), b[:n].view(torch.int32)), n
    cfg = ocfg(**shape)
    w, y = O.windows_at(streams, np.arange(64), np.full(64, W), W)
    o = O.forward(O.init_flat(cfg, 11), cfg, w, y, mode="fp64")
    check_parity("fp32", z[:64].cpu().numpy(), b[:64].cpu().numpy(), o)


@pytest.mark.parametrize("which,n", [(1, 1), (1, 37), (2, 5), (2, 130), (2, 600), ("d256", 17), ("d256", 130)])
def test_small_batch_gradients_match_oracle(which, n):
    """Gradients at batches that are no multiple of the 16-value k-steps, with
    fewer k-steps than waves, with 16- and 32-wide tiles and with the tall
    products (k = n T) split over blocks: the fp32 bar of the update."""
    shape = _shape(which)
    cfg = ocfg(**shape)
    W = shape["W"]
    streams = synth.random_streams(21, n, W + 4)
    s = to_dev(streams)
    flat = synth.random_flat(5, O.init_flat(cfg, 1).size, 0.05)
    m = make_model(shape, "fp32", 0, max_windows=n, max_keep=n, flat=flat)
    m.forward_bits(s, W + 2, 1, keep=True)
    m.adapt_step()
    got = O.unflatten(m.grads(), cfg)
    w, y = O.windows_at(streams, np.arange(n), np.full(n, W + 2), W)
    _, ref = O.forward_backward(flat, cfg, w, y, mode="fp64")
    for k, r in ref.items():
        err = np.abs(got[k] - r) - (1e-4 * np.abs(r) + 1e-5 * np.abs(r).max())
        assert err.max() <= 0, (k, float(err.max()))
