"""The acceptance scan where its division can go wrong: rows that begin anywhere in a 16-byte vector, rows shorter than
one, chunk counts around a chunk and around a workgroup's run, runs of whole rows, more runs than workgroups; both rules,
all logit types, against the oracle.  A -inf prefix longer than a run must not disturb the sum."""
import numpy as np
import pytest
import torch

from oracle import s4c_oracle as O
from paper_2506_14158_amd import binding as B, synth
from paper_2506_14158_amd.device import np_to_torch
from paper_2506_14158_amd.verify import TreeVerifier
from tests.util import MARGIN_MIN

pytestmark = pytest.mark.gpu
C = synth.CONFIGS

# (B, N, levels, V, elements that the logits start behind a 16-byte boundary)
SIZES = [(1, 3, 3, 1, 0), (2, 7, 4, 5, 3), (1, 15, 4, 8191, 0), (2, 17, 5, 8192, 1), (3, 33, 6, 8193, 7), (18, 60, 6, 8192, 5),
         (9, 128, 9, 16383, 0), (2, 61, 6, 50257, 1), (4, 60, 6, 128256, 0), (1, 9, 4, 262144, 2)]


@pytest.mark.parametrize("size", SIZES, ids=str)
@pytest.mark.parametrize("dtype", ["bf16", "f16", "f32"])
@pytest.mark.parametrize("mode", ["greedy", "stochastic"])
def test_scan_division(size, dtype, mode):
    Bn, N, levels, V, off = size
    cfg = synth.scaled(C[2 if mode == "greedy" else 3], name="scan", B=Bn, N=N, levels=levels, V=V, dtype=dtype, index=0)
    par = synth.make_parent(cfg)
    ac = synth.make_accept_inputs(cfg, par)
    lg = np_to_torch(ac.logits, "cpu")
    if mode == "greedy" and V > 8:                       # ties and the ends of a row
        lg[:, 1::4, -1] = 60.0
        lg[:, 2::4, 0] = 60.0
        lg[:, 2::4, V // 2] = 60.0
    elif V > 8192:
        lg[:, ::2, :V // 2] = float("-inf")
    host = lg.view(torch.int16).numpy().view(np.uint16) if dtype == "bf16" else lg.numpy()
    r = O.accept_path(host, par, ac.tokens, mode, levels, ac.p_draft, ac.uniforms, cfg.temperature)
    assert mode == "greedy" or float(r["margin"].min()) > MARGIN_MIN        # fp32 and fp64 decide alike
    flat = torch.empty(lg.numel() + off, dtype=lg.dtype, device="cuda")
    dev = flat[off:].view(lg.shape)
    dev.copy_(lg)
    tv = TreeVerifier(Bn, N, 1, 1, 64, 1, V, lg.dtype, levels, 0)
    t = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()
    tv.accept_path(dev, t(par), t(ac.tokens), B.S4C_GREEDY if mode == "greedy" else B.S4C_STOCHASTIC, t(ac.p_draft), t(ac.uniforms), cfg.temperature)
    torch.cuda.synchronize()
    for name, got in (("status", tv.accept_status), ("path", tv.path), ("accept_len", tv.accept_len),
                      ("accepted_tokens", tv.accepted_tokens), ("bonus_token", tv.bonus_token)):
        assert np.array_equal(got.cpu().numpy(), r[name]), name
