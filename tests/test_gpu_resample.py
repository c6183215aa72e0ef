"""GPU-vs-oracle parity of s4c_accept_resample (sibling-sequential rule with the correction
token) through the C ABI: paths, accepted tokens and the correction token bit-exact."""
import os

import numpy as np
import pytest
import torch

from oracle import s4c_oracle as O
from paper_2506_14158_amd import binding as B, synth
from paper_2506_14158_amd.verify import TreeVerifier
from tests.util import resample_inputs_with_margin, to_device, RESAMPLE_MARGIN_MIN
from tests.test_oracle_resample import read_examples, logp

pytestmark = pytest.mark.gpu
C = synth.CONFIGS


def run(cfg, par, ac, max_path=None):
    d = to_device(cfg, par, None, ac)
    tv = TreeVerifier(cfg.B, cfg.N, 1, 1, 64, 1, cfg.V, d["logits"].dtype, cfg.levels if max_path is None else max_path, 0)
    for t in (tv.path, tv.accept_len, tv.accepted_tokens, tv.bonus_token, tv.accept_status):
        t.fill_(-7)
    tv.accept_resample(d["logits"], d["draft_probs"], d["parent"], d["tokens"], d["uniforms"], d["u_resample"],
                       cfg.temperature)
    torch.cuda.synchronize()
    return tv


def same(tv, r):
    assert np.array_equal(tv.accept_status.cpu().numpy(), r["status"])
    assert np.array_equal(tv.accept_len.cpu().numpy(), r["accept_len"])
    assert np.array_equal(tv.path.cpu().numpy(), r["path"])
    assert np.array_equal(tv.accepted_tokens.cpu().numpy(), r["accepted_tokens"])
    assert np.array_equal(tv.bonus_token.cpu().numpy(), r["bonus_token"])


def check(cfg):
    par = synth.make_parent(cfg)
    ac, r = resample_inputs_with_margin(cfg, par, O)
    tv = run(cfg, par, ac)
    same(tv, r)
    return r


SMALL = [
    synth.scaled(C[3], name="13b-small", B=3, V=9000, index=0),
    synth.scaled(C[3], name="13b-temp", B=2, V=9000, temperature=0.7, index=0),
    synth.scaled(C[3], name="13b-v-odd", B=3, V=8191 * 3 + 5, index=0),                   # rows not 16-byte aligned
    synth.scaled(C[3], name="13b-v-tiny", B=4, V=130, index=0),                           # one partial block
    synth.scaled(C[5], name="70b-small", B=2, V=20000, index=0),                          # N = 128
    synth.scaled(C[1], name="f32", mode="stochastic", B=4, V=5000, N=31, levels=5, index=0),
    synth.scaled(C[1], name="f32-v-odd", mode="stochastic", B=2, V=1003, N=15, levels=4, index=0),
    synth.scaled(C[3], name="root-only", B=3, V=4000, N=1, levels=1, index=0),
    synth.scaled(C[3], name="13b-v-1m", B=2, V=1_000_003, N=6, levels=3, index=0),        # long, odd rows; 16 workgroups each
]


@pytest.mark.parametrize("cfg", SMALL, ids=lambda c: c.name)
def test_accept_resample_small(cfg):
    check(cfg)


@pytest.mark.parametrize("idx", [3, 5])
def test_accept_resample_full_size(idx):
    r = check(C[idx])
    print("cfg%d sequential accept_len" % idx, r["accept_len"].tolist(), "correction tokens", r["bonus_token"].tolist())


def test_independent_candidates_many_sequences():
    """Candidates drawn independently from the draft (the setting of the rule's guarantee), small V,
    many rejections and corrections per tree: 2000 sequences against the oracle."""
    rng = np.random.default_rng(21)
    Bn, V = 2000, 48
    par1 = np.array([-1, 0, 0, 0, 1, 1, 2, 2, 3, 4, 4], dtype=np.int32)
    N = len(par1)
    par = np.tile(par1, (Bn, 1))
    logits = (1.5 * rng.standard_normal((Bn, N, V))).astype(np.float32)
    q = rng.dirichlet(np.full(V, 0.5), size=(Bn, N)).astype(np.float32)
    tokens = np.zeros((Bn, N), dtype=np.int32)
    for c in range(1, N):
        cdf = np.cumsum(q[:, par1[c]].astype(np.float64), axis=1)
        tokens[:, c] = np.minimum((cdf < rng.random((Bn, 1)) * cdf[:, -1:]).sum(1), V - 1)
    u = rng.random((Bn, N), dtype=np.float32)
    ur = rng.random(Bn, dtype=np.float32)
    r = O.accept_resample(logits, q, par, tokens, u, ur, 4)
    good = (r["margin_accept"] > RESAMPLE_MARGIN_MIN) & (r["margin_sample"] > RESAMPLE_MARGIN_MIN)
    assert good.mean() > 0.999
    cfg = synth.scaled(C[1], name="iid", mode="stochastic", B=Bn, N=N, V=V, levels=4, index=0)
    ac = synth.AcceptInputs(logits, tokens, np.zeros((Bn, N), np.float32), u, q, ur)
    tv = run(cfg, par, ac)
    for name in ("accept_len", "bonus_token"):
        assert np.array_equal(getattr(tv, name).cpu().numpy()[good], r[name][good])
    assert np.array_equal(tv.path.cpu().numpy()[good], r["path"][good])
    assert (r["accept_len"] > 0).mean() > 0.3 and (r["accept_len"] == 0).mean() > 0.05


@pytest.mark.parametrize("ex", read_examples(), ids=lambda e: e["name"])
def test_hand_examples_on_the_gpu(ex):
    logits = np.stack([logp(ex["pt0"]), logp(ex["pt1"]), logp(ex["pt2"])])[None]
    q = np.zeros((1, 3, 4), dtype=np.float32)
    q[0, 0] = ex["q0"]
    par = np.array([[-1, 0, 0]], dtype=np.int32)
    tokens = np.array([[9, ex["tok"][0], ex["tok"][1]]], dtype=np.int32)
    cfg = synth.scaled(C[1], name="hand", mode="stochastic", B=1, N=3, V=4, levels=3, index=0)
    ac = synth.AcceptInputs(logits, tokens, np.zeros((1, 3), np.float32), np.array([[0.0] + ex["u"]], np.float32), q,
                            np.array([ex["ur"]], np.float32))
    tv = run(cfg, par, ac)
    assert tv.path.cpu().tolist()[0] == ex["path"] + [-1] * (3 - len(ex["path"]))
    assert int(tv.bonus_token[0]) == ex["bonus"] and int(tv.accept_len[0]) == len(ex["path"]) - 1


def test_equality_rejects_bad_tree_and_bad_token():
    # u * q(x) == r(x) exactly: strict test fails on the GPU as in the oracle
    lg = np.zeros((1, 2, 4), np.float32)
    q = np.zeros((1, 2, 4), np.float32)
    q[0, 0] = [0.5, 0.5, 0, 0]
    cfg = synth.scaled(C[1], name="eq", mode="stochastic", B=1, N=2, V=4, levels=2, index=0)
    for uu, want in ((0.5, 0), (0.49999997, 1)):
        ac = synth.AcceptInputs(lg, np.array([[0, 1]], np.int32), np.zeros((1, 2), np.float32),
                                np.array([[0, uu]], np.float32), q, np.array([0.1], np.float32))
        tv = run(cfg, np.array([[-1, 0]], np.int32), ac)
        assert int(tv.accept_len[0]) == want
    # malformed tree -> flagged; token outside the vocabulary -> skipped
    V = 5
    lg = np.zeros((2, 3, V), np.float32)
    q = np.full((2, 3, V), 0.2, np.float32)
    par = np.array([[-1, 0, 0], [-1, 2, 0]], np.int32)
    tokens = np.array([[0, 77, 1], [0, 1, 1]], np.int32)
    u = np.full((2, 3), 0.5, np.float32)
    ur = np.array([0.5, 0.5], np.float32)
    cfg = synth.scaled(C[1], name="bad", mode="stochastic", B=2, N=3, V=V, levels=3, index=0)
    tv = run(cfg, par, synth.AcceptInputs(lg, tokens, np.zeros((2, 3), np.float32), u, q, ur))
    same(tv, O.accept_resample(lg, q, par, tokens, u, ur, 3))
    assert tv.accept_status.cpu().tolist() == [0, 1]


def test_team_that_cannot_exchange_is_flagged_and_every_kernel_exits(monkeypatch):
    """The bounded wait of the workgroup teams, forced from the host: with zero polls allowed a
    workgroup that does not find all of its team's partial sums at its first look gives up, so no
    team of several workgroups completes.  Every kernel must still exit, and every such sequence
    must come back as the flagged empty result (written by the team's first workgroup alone); the
    next call with the default limit gives the oracle's answer again on the same buffers."""
    cfg = synth.scaled(C[3], name="timeout", B=3, V=40000, index=0)          # teams of 10 workgroups
    par = synth.make_parent(cfg)
    ac, r = resample_inputs_with_margin(cfg, par, O)
    assert B.s4c_accept_resample_workspace_size(cfg.B, cfg.N, cfg.V, cfg.levels) > 0    # teams of more than one workgroup
    d = to_device(cfg, par, None, ac)
    tv = TreeVerifier(cfg.B, cfg.N, 1, 1, 64, 1, cfg.V, d["logits"].dtype, cfg.levels, 0)
    call = lambda: tv.accept_resample(d["logits"], d["draft_probs"], d["parent"], d["tokens"], d["uniforms"],
                                      d["u_resample"], cfg.temperature)
    monkeypatch.setenv("S4C_RESAMPLE_SPIN_LIMIT", "0")
    for rep in range(3):
        for t in (tv.path, tv.accept_len, tv.accepted_tokens, tv.bonus_token, tv.accept_status):
            t.fill_(-7)
        call()
        torch.cuda.synchronize()
        assert tv.accept_status.cpu().tolist() == [B.S4C_SEQ_TIMEOUT] * cfg.B, rep
        assert tv.accept_len.cpu().tolist() == [0] * cfg.B and tv.bonus_token.cpu().tolist() == [-1] * cfg.B
        assert tv.path.cpu().tolist() == [[0] + [-1] * (cfg.levels - 1)] * cfg.B
        assert (tv.accepted_tokens.cpu().numpy() == -1).all()
    monkeypatch.delenv("S4C_RESAMPLE_SPIN_LIMIT")
    call()
    torch.cuda.synchronize()
    same(tv, r)


def test_decisions_given_up_on_are_not_left_behind(monkeypatch):
    """One workgroup per node, and the one that follows the decisions gives up at once: none of them may stay in the
    workspace, where a replay of the same captured call would take it for its own."""
    cfg = synth.scaled(C[3], name="timeout-rows", B=3, V=4000, index=0)
    par = synth.make_parent(cfg)
    ac, r = resample_inputs_with_margin(cfg, par, O)
    d = to_device(cfg, par, None, ac)
    tv = TreeVerifier(cfg.B, cfg.N, 1, 1, 64, 1, cfg.V, d["logits"].dtype, cfg.levels, 0)
    call = lambda: tv.accept_resample(d["logits"], d["draft_probs"], d["parent"], d["tokens"], d["uniforms"],
                                      d["u_resample"], cfg.temperature)
    monkeypatch.setenv("S4C_RESAMPLE_SPIN_LIMIT", "0")
    call()
    torch.cuda.synchronize()
    assert tv.accept_status.cpu().tolist() == [B.S4C_SEQ_TIMEOUT] * cfg.B
    words = tv.resample_ws.view(torch.int32)[:2 * cfg.B * cfg.N].cpu().reshape(-1, 2)
    assert (words[:, 0] == 0).all() and (words[:, 1] == words[0, 1]).all()
    monkeypatch.delenv("S4C_RESAMPLE_SPIN_LIMIT")
    call()
    torch.cuda.synchronize()
    same(tv, r)


def test_rejects_bad_arguments():
    t = lambda *s, dt=torch.float32: torch.zeros(*s, dtype=dt, device="cuda")
    i = lambda *s: torch.zeros(*s, dtype=torch.int32, device="cuda")
    with pytest.raises(B.S4CError):      # temperature must be positive
        B.s4c_accept_resample(t(1, 2, 8), t(1, 2, 8), i(1, 2), i(1, 2), t(1, 2), t(1), 2, i(1, 2), i(1), i(1, 2), i(1),
                              temperature=0.0)
    with pytest.raises(B.S4CError):      # a team of workgroups needs its exchange workspace
        assert B.s4c_accept_resample_workspace_size(2, 3, 40000, 3) > 0
        B.s4c_accept_resample(t(2, 3, 40000), t(2, 3, 40000), i(2, 3), i(2, 3), t(2, 3), t(2), 3, i(2, 3), i(2), i(2, 3),
                              i(2), workspace=None)
    with pytest.raises(B.S4CError):      # more nodes than a tree may hold
        B.s4c_accept_resample(t(1, 129, 8), t(1, 129, 8), i(1, 129), i(1, 129), t(1, 129), t(1), 2, i(1, 2), i(1),
                              i(1, 2), i(1))


def random_call(Bn, N, V, dtype):
    """Inputs of a call on the device, their type, the tree's levels, and what the oracle says."""
    levels = min(N, 5)
    par = np.stack([synth.random_tree_parent(N, levels, (8, 4, 3, 2, 2), np.random.default_rng([7, b])) for b in range(Bn)]).astype(np.int32)
    g = torch.Generator().manual_seed(V + N)
    dt = {"f32": torch.float32, "bf16": torch.bfloat16, "f16": torch.float16}[dtype]
    logits = (2 * torch.randn(Bn, N, V, generator=g)).to(dt)
    pd = torch.softmax(logits.float() + 0.5 * torch.randn(Bn, N, V, generator=g), 2)
    top = pd.topk(min(8, V), 2).indices
    tokens = torch.zeros(Bn, N, dtype=torch.int32)
    for b in range(Bn):
        for i in range(1, N):
            rank = sum(1 for j in range(1, i) if par[b, j] == par[b, i])
            tokens[b, i] = top[b, par[b, i], min(rank, top.shape[2] - 1)]
    u, ur = torch.rand(Bn, N, generator=g), torch.rand(Bn, generator=g)
    u[0] = 0.9999                                        # (sequence 0 rejects nearly everything)
    bits = lambda t: t.numpy() if dtype == "f32" else t.view(torch.int16).numpy().view(np.uint16) if dtype == "bf16" else t.numpy()
    r = O.accept_resample(bits(logits), pd.numpy(), par, tokens.numpy(), u.numpy(), ur.numpy(), levels)
    assert min(float(r["margin_accept"].min()), float(r["margin_sample"].min())) > RESAMPLE_MARGIN_MIN
    return [t.cuda() for t in (logits, pd, torch.from_numpy(par), tokens, u, ur)], dt, levels, r


@pytest.mark.parametrize("Bn,N,V,dtype", [(2, 20, 1, "bf16"), (1, 2, 4095, "f32"), (3, 33, 4097, "bf16"), (5, 64, 8193, "f16"),
                                          (2, 40, 16384, "f32"), (2, 40, 16385, "bf16"), (2, 12, 32768, "f16"), (2, 12, 32769, "bf16"),
                                          (1, 9, 65544, "f32"), (2, 5, 524289, "bf16"), (129, 3, 8000, "bf16"),
                                          (40, 4, 128256, "bf16")])
def test_one_workgroup_per_node_teams_and_replays(Bn, N, V, dtype):
    """Block, register and route edges.  The same call decides every node at once where rows are few and short, or
    walks with teams; it does without a workspace where a workgroup a sequence is enough, and replays from a captured graph; all of them as the oracle."""
    d, dt, levels, r = random_call(Bn, N, V, dtype)
    tv = TreeVerifier(Bn, N, 1, 1, 64, 1, V, dt, levels, 0)
    outs = (tv.path, tv.accept_len, tv.accepted_tokens, tv.bonus_token, tv.accept_status)

    def call(ws):
        for t in outs:
            t.fill_(-7)
        B.s4c_accept_resample(*d, levels, tv.path, tv.accept_len, tv.accepted_tokens, tv.bonus_token, ws, 1.0, tv.accept_status)
        torch.cuda.synchronize()
        same(tv, r)

    for t in (0xFF, 0x00):                               # whatever the workspace holds
        tv.resample_ws.fill_(t)
        call(tv.resample_ws)
    if V <= 4096 or Bn > 128:
        call(None)                                       # one workgroup per sequence needs no workspace
        call(tv.resample_ws[:8])                         # (too small for a word per node)
    gr = torch.cuda.CUDAGraph()
    with torch.cuda.graph(gr):
        tv.accept_resample(*d, 1.0)
    for _ in range(4):
        for t in outs:
            t.fill_(-7)
        gr.replay()
        torch.cuda.synchronize()
        same(tv, r)


def test_more_sequences_than_a_launch_of_teams_takes():
    """130 teams of 2: 128 in a launch, and the last two in one that is filled up with workgroups without a sequence."""
    d, dt, levels, r = random_call(130, 2, 33000, "bf16")
    tv = TreeVerifier(130, 2, 1, 1, 64, 1, 33000, dt, levels, 0)
    for _ in range(2):
        for t in (tv.path, tv.accept_len, tv.accepted_tokens, tv.bonus_token, tv.accept_status):
            t.fill_(-7)
        tv.accept_resample(*d, 1.0)
        torch.cuda.synchronize()
        same(tv, r)


def test_calls_on_two_streams():
    """Each call's teams take the chip's CUs one by one (40 x 4 slices of 32768) or two to a CU (16 x 16 of 8192), with a workspace
    of its own; together they complete."""
    calls = []
    for Bn, N, V in ((40, 4, 128256), (16, 10, 128256), (33, 5, 128256)):
        d, dt, levels, r = random_call(Bn, N, V, "bf16")
        calls.append((TreeVerifier(Bn, N, 1, 1, 64, 1, V, dt, levels, 0), d, r))
    streams = [torch.cuda.Stream(), torch.cuda.Stream()]
    torch.cuda.synchronize()
    for i, k in ((0, 1), (0, 2), (1, 2)):
        for c, st in ((calls[i], streams[0]), (calls[k], streams[1])):
            with torch.cuda.stream(st):
                for _ in range(5):
                    c[0].accept_resample(*c[1], 1.0)
        torch.cuda.synchronize()
        for tv, _, r in (calls[i], calls[k]):
            same(tv, r)
            for t in (tv.path, tv.accept_len, tv.accepted_tokens, tv.bonus_token, tv.accept_status):
                t.fill_(-7)
