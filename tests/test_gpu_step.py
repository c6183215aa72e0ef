"""s4c_verify_step (TreeVerifier.step) against the three calls it replaces, every output bit for bit: divided and
undivided attention, KV head counts around the number of copying workgroups, sequences that do not fit the cache, a
malformed tree, logits of another type than the cache (three launches), several calls on one workspace."""
import numpy as np
import pytest
import torch

from paper_2506_14158_amd import synth
from paper_2506_14158_amd.verify import TreeVerifier
from tests.util import to_device

pytestmark = pytest.mark.gpu
C = synth.CONFIGS

CASES = [
    synth.scaled(C[1], name="tiny", index=0),
    synth.scaled(C[2], name="7b-parts", Hq=9, Hkv=9, P=1500, V=9000, index=0),                        # 9 heads: two per copier
    synth.scaled(C[3], name="13b-one-head", B=3, Hq=1, Hkv=1, P=333, V=32000, ragged=True, index=0),
    synth.scaled(C[4], name="gqa", B=2, Hq=16, Hkv=4, P=700, V=70001, index=0),                       # rows not 16-byte aligned
    synth.scaled(C[5], name="70b", B=2, Hq=16, Hkv=2, P=3000, V=20000, ragged=True, index=0),
    synth.scaled(C[3], name="d64-f16", B=3, Hq=12, Hkv=12, D=64, P=500, V=9000, dtype="f16", index=0),
]


@pytest.mark.parametrize("cfg", CASES, ids=lambda c: c.name)
@pytest.mark.parametrize("logits", ["same", "f32"])
def test_step_equals_the_three_calls(cfg, logits):
    par = synth.make_parent(cfg)
    if cfg.B >= 3:
        par[1, 1] = 5                                       # a node before its parent: flagged everywhere
    at, ac = synth.make_attn_inputs(cfg), synth.make_accept_inputs(cfg, synth.make_parent(cfg))
    d = to_device(cfg, par, at, ac)
    if logits == "f32":
        d["logits"] = d["logits"].float()
    S_cap = cfg.P + 1                                       # room for one row: longer paths do not fit
    kc, vc = d["k_cache"][:, :, :S_cap].contiguous(), d["v_cache"][:, :, :S_cap].contiguous()
    mode = 0 if cfg.mode == "greedy" else 1
    seen = []
    for fused in (True, True, False):
        tv = TreeVerifier(cfg.B, cfg.N, cfg.Hq, cfg.Hkv, cfg.D, S_cap, cfg.V, d["q"].dtype, cfg.levels, cfg.P)
        k, v, n = kc.clone(), vc.clone(), d["cache_len"].clone()
        rest = (d["logits"], d["tokens"], mode, d["p_draft"], d["uniforms"], cfg.temperature)
        for _ in range(2):                                  # the second step reads what the first appended
            n.clamp_(max=cfg.P)
            if fused:
                tv.step(d["q"], d["k_tree"], d["v_tree"], k, v, n, d["parent"], *rest)
            else:
                tv.tree_attn(d["q"], d["k_tree"], d["v_tree"], k, v, n, d["parent"])
                tv.accept_path(rest[0], d["parent"], *rest[1:])
                tv.kv_compact(d["k_tree"], d["v_tree"], k, v, n)
        torch.cuda.synchronize()
        seen.append([t.clone() for t in (tv.out, tv.path, tv.accept_len, tv.accepted_tokens, tv.bonus_token, tv.dst_index,
                                         tv.attn_status, tv.accept_status, tv.compact_status, k, v, n)])
    for other in seen[1:]:
        for x, y in zip(seen[0], other):
            assert torch.equal(x.view(torch.uint8), y.view(torch.uint8))
    if cfg.B >= 3:
        assert int(seen[0][7][1]) != 0


def test_a_copier_that_gives_up_flags_the_sequence_and_leaves_its_length(monkeypatch):
    """The bounded wait of the workgroups that append the rows, forced from the host: with a waiting time of zero one that does
    not find its message at its first look leaves.  All workgroups of these launches fit on the GPU at once, so the copiers
    look while the scan has 300 KB a row still to read, of which the message is a consequence.  The path is right all the same,
    the sequences are flagged, their lengths and caches untouched, also when a captured graph repeats the call (whose nonce is
    that of the message nobody took); with the usual wait the same buffers then give what the three calls give, and so does a graph."""
    cfg = synth.scaled(C[4], name="copier-timeout", B=2, Hq=8, Hkv=4, P=200, N=8, levels=4, V=150_007, index=0)
    par = synth.make_parent(cfg)
    at, ac = synth.make_attn_inputs(cfg), synth.make_accept_inputs(cfg, par)
    d = to_device(cfg, par, at, ac)
    tv = TreeVerifier(cfg.B, cfg.N, cfg.Hq, cfg.Hkv, cfg.D, cfg.S_cap, cfg.V, d["q"].dtype, cfg.levels, cfg.P)
    k, v, n = d["k_cache"].clone(), d["v_cache"].clone(), d["cache_len"].clone()
    rest = (d["logits"], d["tokens"], 0)
    step = lambda: tv.step(d["q"], d["k_tree"], d["v_tree"], k, v, n, d["parent"], *rest)
    outputs = lambda: [t.clone() for t in (tv.out, tv.path, tv.accept_len, tv.accepted_tokens, tv.bonus_token, tv.accept_status)]

    def reset():
        for dst, src in ((k, "k_cache"), (v, "v_cache"), (n, "cache_len")):
            dst.copy_(d[src])
        for t in (tv.path, tv.accept_len, tv.dst_index, tv.compact_status):
            t.fill_(-7)
        torch.cuda.synchronize()

    def captured():
        g, side = torch.cuda.CUDAGraph(), torch.cuda.Stream()
        with torch.cuda.stream(side):
            with torch.cuda.graph(g, stream=side):
                step()
        return g.replay

    same = lambda a, b: all(torch.equal(x.view(torch.uint8), y.view(torch.uint8)) for x, y in zip(a, b))
    reset()
    tv.tree_attn(d["q"], d["k_tree"], d["v_tree"], k, v, n, d["parent"])
    tv.accept_path(d["logits"], d["parent"], *rest[1:])
    tv.kv_compact(d["k_tree"], d["v_tree"], k, v, n)
    torch.cuda.synchronize()
    want, appended = outputs(), [t.clone() for t in (k, v, n, tv.dst_index, tv.compact_status)]

    monkeypatch.setenv("S4C_COPY_WAIT_US", "0")
    for call in [step] + [captured()] * 3:
        reset()
        call()
        torch.cuda.synchronize()
        assert tv.compact_status.tolist() == [4] * cfg.B                       # S4C_SEQ_TIMEOUT
        assert (tv.dst_index == -1).all() and same([k, v, n], [d["k_cache"], d["v_cache"], d["cache_len"]])
        assert same(outputs(), want)
    monkeypatch.delenv("S4C_COPY_WAIT_US")
    for call in [step] + [captured()] * 3:
        reset()
        call()
        torch.cuda.synchronize()
        assert same(outputs(), want) and same([k, v, n, tv.dst_index, tv.compact_status], appended)
