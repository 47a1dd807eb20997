"""The attention kernel of bf16 launches over runs of positions (byte groups
shared between the 64 windows of a tile, one stream per tile), for every shape it
is built for: runs that end inside a tile, chunks that cut tiles, both workgroup
sizes, against the per-token kernel and the oracle."""
import numpy as np
import pytest
import torch

import oracle as O
import synth
from gpu_helpers import check_parity, make_model, ocfg, to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("D,DH", [(128, 32), (256, 32), (256, 64), (512, 64)])
@pytest.mark.parametrize("T,g", [(8, 8), (8, 4), (4, 8), (4, 4)])
def test_runs_match_token_kernel_and_oracle(D, DH, T, g):
    W = T * g
    shape = dict(W=W, e=D // g, g=g, H=D // DH, F=256, k=1)
    cfg = ocfg(**shape)
    flat = synth.random_flat(3, O.init_flat(cfg, 1).size, 0.06)
    B, S = 5, 131
    streams = synth.random_streams(17, B, W + 3 + S)
    s = to_dev(streams)
    m = make_model(shape, "bf16", 0, max_windows=1 << 16, flat=flat)
    # 40: less than a tile; 64, 65: at and past its edge; 131: three tiles, the last of 3
    for n in (40, 64, 65, S):
        pos0 = W + 3
        r = m.forward_bits(s, pos0, n, logits=True)
        t = m.forward_bits(s, pos0, n, logits=True, token_attn=True)
        z, zt = r["logits"].double(), t["logits"].double()
        # two sum orders over the same bf16 storage points: within the forward's bf16 bar
        rel = (z - zt).abs().amax(1) / zt.abs().amax(1)
        assert float(rel.max()) <= 2e-2, (n, float(rel.max()))
        # chunks of 37 windows cut tiles anywhere: the same bits
        mc = make_model(shape, "bf16", 0, max_windows=37, flat=flat)
        c = mc.forward_bits(s, pos0, n, logits=True)
        assert torch.equal(c["logits"].view(torch.int32), r["logits"].view(torch.int32)), n
    b, i = synth.sample_positions(5, B, W + 3 + S, W + 3, 96)
    w, y = O.windows_at(streams, b, i, W)
    ref = O.forward(flat, cfg, w, y, mode="bf16")
    idx = torch.from_numpy(b * S + (i - W - 3)).cuda()
    check_parity("bf16", r["logits"][idx].cpu().numpy(), r["bits"][idx].cpu().numpy(), ref)
    # more tiles than CUs (the other workgroup size), each stream the same bytes
    many = s[:1].repeat(300, 1).contiguous()
    z = m.forward_bits(many, W + 3, 40, logits=True)["logits"].view(300, 40, 256)
    assert torch.equal(z.view(torch.int32), z[:1].expand_as(z).contiguous().view(torch.int32))
    one = m.forward_bits(s[:1].contiguous(), W + 3, 40, logits=True)["logits"]
    assert torch.equal(z[7].view(torch.int32), one.view(torch.int32))
