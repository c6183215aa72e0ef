"""A step in one launch, and divided attention merged in its own: against the oracle and the separate calls, eagerly and from a captured
graph, where the attention leaves few places, sequences have fewer copiers, and several calls overlap."""
import numpy as np
import pytest
import torch

from oracle import s4c_oracle as O
from paper_2506_14158_amd import synth
from paper_2506_14158_amd.verify import TreeVerifier
from tests.util import attn_errors, to_device

pytestmark = pytest.mark.gpu
C = synth.CONFIGS
TOL = {"f32": (1e-5, 1e-5), "bf16": (1e-2, 2e-2), "f16": (2e-3, 4e-3)}      # the storage type's rounding of P and of the output, as in the parity tests

CASES = [
    synth.scaled(C[3], name="most-places", B=4, Hq=40, Hkv=40, P=2000, V=4000, index=0),                 # 480 workgroups attend
    synth.scaled(C[3], name="32-sequences", B=32, Hq=5, Hkv=5, P=300, N=20, levels=5, V=2000, ragged=True, index=0),     # two copiers each
    synth.scaled(C[2], name="odd-f16", B=3, Hq=7, Hkv=7, P=777, N=33, levels=5, V=5003, dtype="f16", ragged=True, index=0),
    synth.scaled(C[1], name="f32-d64", B=2, Hq=3, Hkv=3, P=900, N=17, V=3001, index=0),
    synth.scaled(C[5], name="many-rows", B=1, Hq=32, Hkv=4, P=2000, N=60, levels=6, V=9001, index=0),
    synth.scaled(C[4], name="80-rows-d64", B=2, Hq=10, Hkv=5, D=64, P=1500, N=40, levels=6, V=6000, index=0),
]


def _in_one_launch(tv, run):
    """Whether `run` left marks where a step of one launch has its attention workgroups tell that they have read the lengths."""
    words = tv.accept_ws[-tv.B * torch.cuda.get_device_properties(0).multi_processor_count * 2 * 16:]
    words.fill_(0x5A)
    run()
    torch.cuda.synchronize()
    return bool((words != 0x5A).any())


def _same(a, b):
    return all(torch.equal(x.contiguous().view(torch.uint8), y.contiguous().view(torch.uint8)) for x, y in zip(a, b))


@pytest.mark.parametrize("cfg", CASES, ids=lambda c: c.name)
def test_eager_and_replayed_steps(cfg):
    par = synth.make_parent(cfg)
    at, ac = synth.make_attn_inputs(cfg), synth.make_accept_inputs(cfg, par)
    d = to_device(cfg, par, at, ac)
    mode = 0 if cfg.mode == "greedy" else 1
    tv = TreeVerifier(cfg.B, cfg.N, cfg.Hq, cfg.Hkv, cfg.D, cfg.S_cap, cfg.V, d["q"].dtype, cfg.levels, cfg.P)
    k, v, n = d["k_cache"].clone(), d["v_cache"].clone(), d["cache_len"].clone()
    rest = (d["logits"], d["tokens"], mode, d["p_draft"], d["uniforms"], cfg.temperature)
    step = lambda: tv.step(d["q"], d["k_tree"], d["v_tree"], k, v, n, d["parent"], *rest)
    seen = lambda: [t.clone() for t in (tv.out, tv.path, tv.accept_len, tv.accepted_tokens, tv.bonus_token, tv.dst_index, tv.attn_status,
                                        tv.accept_status, tv.compact_status, k, v, n)]

    def reset():
        for dst, src in ((k, "k_cache"), (v, "v_cache"), (n, "cache_len")):
            dst.copy_(d[src])
        tv.out.fill_(7.0)

    reset()
    assert _in_one_launch(tv, step)
    assert (tv.num_splits > 1) == (cfg.name != "32-sequences")
    first = seen()
    ref, _ = O.tree_attn(at.q, at.k_tree, at.v_tree, at.k_cache, at.v_cache, at.cache_len, par)
    amax, rel = attn_errors(tv.out, ref)
    assert amax <= TOL[cfg.dtype][0] and rel <= TOL[cfg.dtype][1], (amax, rel)
    r = O.accept_path(ac.logits, par, ac.tokens, cfg.mode, cfg.levels, ac.p_draft, ac.uniforms, cfg.temperature)
    assert np.array_equal(tv.path.cpu().numpy(), r["path"]) and np.array_equal(tv.accept_len.cpu().numpy(), r["accept_len"])
    kc, vc, cl = at.k_cache.copy(), at.v_cache.copy(), at.cache_len.copy()
    O.kv_compact(at.k_tree, at.v_tree, kc, vc, cl, r["path"], r["accept_len"])
    assert np.array_equal(n.cpu().numpy(), cl)
    assert np.array_equal(k.cpu().contiguous().view(torch.uint8).numpy(), kc.view(np.uint8))
    assert np.array_equal(v.cpu().contiguous().view(torch.uint8).numpy(), vc.view(np.uint8))
    g, side = torch.cuda.CUDAGraph(), torch.cuda.Stream()
    with torch.cuda.stream(side):
        with torch.cuda.graph(g, stream=side):
            step()
    for call in (g.replay, g.replay, step, g.replay):
        reset()
        torch.cuda.synchronize()
        call()
        torch.cuda.synchronize()
        assert _same(seen(), first)


def test_waits_that_run_out_leave_nothing_behind(monkeypatch):
    """A waiting time of zero: collectors that find a length unread, and copiers without a message, flag their sequence and leave its length; so
    does every replay of the call, and the paths are right all the same.  With the usual wait the same workspaces serve again."""
    cfg = synth.scaled(C[4], name="no-wait", B=3, Hq=16, Hkv=8, P=500, N=24, levels=5, V=150_007, index=0)
    par = synth.make_parent(cfg)
    d = to_device(cfg, par, synth.make_attn_inputs(cfg), synth.make_accept_inputs(cfg, par))
    tv = TreeVerifier(cfg.B, cfg.N, cfg.Hq, cfg.Hkv, cfg.D, cfg.S_cap, cfg.V, d["q"].dtype, cfg.levels, cfg.P)
    k, v, n = d["k_cache"].clone(), d["v_cache"].clone(), d["cache_len"].clone()
    step = lambda: tv.step(d["q"], d["k_tree"], d["v_tree"], k, v, n, d["parent"], d["logits"], d["tokens"], 0)
    seen = lambda: [t.clone() for t in (tv.out, tv.path, tv.accept_len, tv.bonus_token)]

    def reset(shorter=0):
        for dst, src in ((k, "k_cache"), (v, "v_cache"), (n, "cache_len")):
            dst.copy_(d[src])
        n.sub_(shorter)
        torch.cuda.synchronize()

    reset()
    assert _in_one_launch(tv, step)
    want, after = seen(), [t.clone() for t in (k, v, n, tv.dst_index, tv.compact_status)]
    monkeypatch.setenv("S4C_COPY_WAIT_US", "0")
    g, side = torch.cuda.CUDAGraph(), torch.cuda.Stream()
    with torch.cuda.stream(side):
        with torch.cuda.graph(g, stream=side):
            step()
    monkeypatch.delenv("S4C_COPY_WAIT_US")
    for i in range(6):
        reset(shorter=7 * (i % 2))
        g.replay()
        torch.cuda.synchronize()
        assert tv.compact_status.tolist() == [4] * cfg.B and bool((tv.dst_index == -1).all())      # S4C_SEQ_TIMEOUT
        assert torch.equal(n, d["cache_len"] - 7 * (i % 2))
        assert _same(seen()[1:], want[1:]) and (i % 2 == 1 or torch.equal(tv.out, want[0]))
    reset()
    step()
    torch.cuda.synchronize()
    assert _same(seen(), want) and _same([k, v, n, tv.dst_index, tv.compact_status], after)


def test_a_step_whose_scan_would_outlast_the_attention_takes_two_launches():
    """Many short rows for the few workgroups that fit beside the attention (tests/test_step_plan.py)."""
    cfg = synth.scaled(C[4], name="short-rows", B=6, Hq=32, Hkv=32, N=69, levels=6, P=134, V=4127, index=0)
    par = synth.make_parent(cfg)
    d = to_device(cfg, par, synth.make_attn_inputs(cfg), synth.make_accept_inputs(cfg, par))
    tv = TreeVerifier(cfg.B, cfg.N, cfg.Hq, cfg.Hkv, cfg.D, cfg.S_cap, cfg.V, d["q"].dtype, cfg.levels, cfg.P)
    k, v, n = d["k_cache"].clone(), d["v_cache"].clone(), d["cache_len"].clone()
    assert not _in_one_launch(tv, lambda: tv.step(d["q"], d["k_tree"], d["v_tree"], k, v, n, d["parent"], d["logits"], d["tokens"], 0))
    seen = [t.clone() for t in (tv.out, tv.path, tv.accept_len, tv.bonus_token, k, v, n)]
    k, v, n = d["k_cache"].clone(), d["v_cache"].clone(), d["cache_len"].clone()
    tv.tree_attn(d["q"], d["k_tree"], d["v_tree"], k, v, n, d["parent"])
    tv.accept_path(d["logits"], d["parent"], d["tokens"], 0)
    tv.kv_compact(d["k_tree"], d["v_tree"], k, v, n)
    torch.cuda.synchronize()
    assert _same(seen, [tv.out, tv.path, tv.accept_len, tv.bonus_token, k, v, n])


@pytest.mark.parametrize("cfg", [CASES[0], CASES[3], CASES[4]], ids=lambda c: c.name)
def test_replayed_attention_reads_the_inputs_of_the_replay(cfg):
    """A part of the replay before has the same tag: new queries between the replays, every result as an eager call gives it."""
    par = synth.make_parent(cfg)
    d = to_device(cfg, par, synth.make_attn_inputs(cfg), synth.make_accept_inputs(cfg, par))
    tv = TreeVerifier(cfg.B, cfg.N, cfg.Hq, cfg.Hkv, cfg.D, cfg.S_cap, cfg.V, d["q"].dtype, cfg.levels, cfg.P)
    assert tv.num_splits > 1
    q = d["q"].clone()
    call = lambda: tv.tree_attn(q, d["k_tree"], d["v_tree"], d["k_cache"], d["v_cache"], d["cache_len"], d["parent"])
    call()
    torch.cuda.synchronize()
    g, side = torch.cuda.CUDAGraph(), torch.cuda.Stream()
    with torch.cuda.stream(side):
        with torch.cuda.graph(g, stream=side):
            call()
    for i in range(6):
        q.copy_(torch.roll(d["q"], i + 1, 0 if cfg.B > 1 else 1) * (1.0 if i % 2 else -1.0))
        call()
        torch.cuda.synchronize()
        want = tv.out.clone()
        tv.out.fill_(7.0)
        tv.attn_status.fill_(7)
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        assert int(tv.attn_status.abs().sum()) == 0 and torch.equal(tv.out, want)


def test_divided_attention_on_four_streams():
    """Four calls at a time, each with its own buffers, whose workgroups fill the chip several times over: some start when others of their
    unit are through.  What each gives by itself, eagerly and replayed."""
    cases = [synth.scaled(C[4], name="a", B=8, Hq=32, Hkv=8, P=2000, V=500, index=0), synth.scaled(C[3], name="b", B=4, Hq=40, Hkv=40, P=1100, V=500, index=0),
             synth.scaled(C[4], name="c", B=13, Hq=32, Hkv=8, N=18, levels=6, P=1500, V=500, index=0),
             synth.scaled(C[1], name="d", B=2, Hq=3, Hkv=3, P=900, N=17, V=500, index=0)]
    runs = []
    for cfg in cases:
        par = synth.make_parent(cfg)
        d = to_device(cfg, par, synth.make_attn_inputs(cfg), synth.make_accept_inputs(cfg, par))
        tv = TreeVerifier(cfg.B, cfg.N, cfg.Hq, cfg.Hkv, cfg.D, cfg.S_cap, cfg.V, d["q"].dtype, cfg.levels, cfg.P)
        assert tv.num_splits > 1

        def call(d=d, tv=tv):
            tv.tree_attn(d["q"], d["k_tree"], d["v_tree"], d["k_cache"], d["v_cache"], d["cache_len"], d["parent"])

        call()
        torch.cuda.synchronize()
        stream, g = torch.cuda.Stream(), torch.cuda.CUDAGraph()
        with torch.cuda.stream(stream):
            with torch.cuda.graph(g, stream=stream):
                call()
        runs.append((call, g.replay, tv, tv.out.clone(), stream))
    torch.cuda.synchronize()
    for i in range(30):
        for call, replay, _, _, stream in runs:
            with torch.cuda.stream(stream):
                call() if i % 2 else replay()
        if i % 10 == 9:
            torch.cuda.synchronize()
            for _, _, tv, alone, _ in runs:
                assert int(tv.attn_status.abs().sum()) == 0 and torch.equal(tv.out, alone)
                tv.out.fill_(7.0)
            torch.cuda.synchronize()


def test_steps_on_four_streams():
    """Four steps that overlap, each with its own buffers: what each gives by itself."""
    runs = []
    for cfg in (CASES[0], CASES[4], CASES[1], CASES[2]):
        par = synth.make_parent(cfg)
        d = to_device(cfg, par, synth.make_attn_inputs(cfg), synth.make_accept_inputs(cfg, par))
        tv = TreeVerifier(cfg.B, cfg.N, cfg.Hq, cfg.Hkv, cfg.D, cfg.S_cap, cfg.V, d["q"].dtype, cfg.levels, cfg.P)
        k, v, n = d["k_cache"].clone(), d["v_cache"].clone(), d["cache_len"].clone()

        def step(d=d, tv=tv, k=k, v=v, n=n, cfg=cfg):
            n.copy_(d["cache_len"])
            tv.step(d["q"], d["k_tree"], d["v_tree"], k, v, n, d["parent"], d["logits"], d["tokens"], 0 if cfg.mode == "greedy" else 1,
                    d["p_draft"], d["uniforms"], cfg.temperature)

        seen = lambda tv=tv, k=k, v=v, n=n: [t.clone() for t in (tv.out, tv.path, tv.accept_len, tv.attn_status, tv.accept_status,
                                                                 tv.compact_status, k, v, n)]
        step()
        torch.cuda.synchronize()
        runs.append((step, seen, seen(), torch.cuda.Stream()))
    torch.cuda.synchronize()
    for _ in range(20):
        for step, _, _, stream in runs:
            with torch.cuda.stream(stream):
                step()
    torch.cuda.synchronize()
    for _, seen, alone, _ in runs:
        assert _same(seen(), alone)
