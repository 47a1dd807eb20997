"""The attention kernel of launches over runs of positions (byte groups shared
between the 64 windows of a tile, one stream per tile), for every shape it is
built for: runs that end inside a tile, chunks that cut tiles, few tiles and
many, against the per-token kernel and the oracle."""
import numpy as np
import pytest
import torch

import oracle as O
import synth
from gpu_helpers import check_parity, make_model, ocfg, oracle_mode, to_dev

pytestmark = pytest.mark.gpu

SHAPES = ([("bf16", D, DH) for D, DH in [(128, 32), (128, 64), (256, 32), (256, 64), (512, 64)]] +
          [("fp32", D, DH) for D, DH in [(64, 32), (64, 64), (128, 32), (128, 64), (256, 32), (256, 64)]])


@pytest.mark.parametrize("dtype,D,DH", SHAPES)
@pytest.mark.parametrize("T,g", [(8, 8), (8, 4), (4, 8), (4, 4)])
def test_runs_match_token_kernel_and_oracle(dtype, D, DH, T, g):
    W = T * g
    shape = dict(W=W, e=D // g, g=g, H=D // DH, F=256, k=1)
    cfg = ocfg(**shape)
    flat = synth.random_flat(3, O.init_flat(cfg, 1).size, 0.06)
    B, S, pos0 = 5, 131, W + 3
    base = synth.random_streams(17, B, pos0 + S)
    # narrow models take this kernel from some thousand windows on: the same streams again
    R = {64: 125, 128: 32}.get(D, 1)
    s = to_dev(np.tile(base, (R, 1)))
    m = make_model(shape, dtype, 0, max_windows=1 << 17, flat=flat)
    # 40: less than a tile; 64, 65: at and past its edge; 131: three tiles, the last of 3
    for n in (40, 64, 65, S):
        r = m.forward_bits(s, pos0, n, logits=True)
        t = m.forward_bits(s, pos0, n, logits=True, token_attn=True)
        z, zt = r["logits"].double(), t["logits"].double()
        # two sum orders over the same storage points: within the forward's bars
        rel = (z - zt).abs().amax(1) / zt.abs().amax(1)
        assert float(rel.max()) <= (2e-2 if dtype == "bf16" else 1e-4), (n, float(rel.max()))
        # a window's result does not depend on its tile: every copy of a stream agrees,
        # and so do chunks of 37 windows, which cut tiles anywhere
        bits = r["logits"].view(torch.int32).view(R, B * n, 256)
        assert torch.equal(bits, bits[:1].expand_as(bits)), n
        mc = make_model(shape, dtype, 0, max_windows=37, flat=flat)
        c = mc.forward_bits(s, pos0, n, logits=True)
        assert torch.equal(c["logits"].view(torch.int32), r["logits"].view(torch.int32)), n
    b, i = synth.sample_positions(5, B, pos0 + S, pos0, 96)
    w, y = O.windows_at(base, b, i, W)
    ref = O.forward(flat, cfg, w, y, mode=oracle_mode(dtype))
    idx = torch.from_numpy(b * S + (i - pos0)).cuda()
    check_parity(dtype, r["logits"][idx].cpu().numpy(), r["bits"][idx].cpu().numpy(), ref)
    if R == 1:  # more tiles than CUs: the other workgroup size, the same bits
        many = m.forward_bits(s[:1].repeat(300, 1), pos0, 40, logits=True)["logits"].view(300, 40, 256)
        one = m.forward_bits(s[:1].contiguous(), pos0, 40, logits=True)["logits"].view(1, 40, 256)
        assert torch.equal(many.view(torch.int32), one.expand_as(many).contiguous().view(torch.int32))
