"""Errors that arise while the native half of the binding reads its arguments are Python exceptions.  No GPU: fake tensors
pass for device tensors until the stream is asked for, which throws where there is no device."""
import pytest
import torch
from torch._subclasses.fake_tensor import FakeTensorMode

from paper_2506_14158_amd import binding as B
from paper_2506_14158_amd.verify import TreeVerifier

Bn, N, H, D, S, V, L, PAGE, LY = 2, 8, 2, 64, 128, 500, 4, 64, 3


def tensors():
    t = lambda *s, dt=torch.bfloat16: torch.empty(*s, dtype=dt, device="cuda")
    i = lambda *s: t(*s, dt=torch.int32)
    f = lambda *s: t(*s, dt=torch.float32)
    return dict(q=t(Bn, N, H, D), tree=t(Bn, N, H, D), cache=t(Bn, H, S, D), pool=t(4, H, PAGE, D), table=i(Bn, S // PAGE), n=i(Bn),
                parent=i(Bn, N), logits=t(Bn, N, V), tokens=i(Bn, N), u=f(Bn, N), u1=f(Bn), dp=f(Bn, N, V), trees=t(LY, Bn, N, H, D),
                caches=t(LY, Bn, H, S, D), pools=t(LY, 4, H, PAGE, D), e=t(4, 256), W=t(256, 512), ws=t(1 << 20, dt=torch.uint8),
                level=i(Bn, N))


CALLS = {
    "tree_attn": lambda v, x: v.tree_attn(x.q, x.tree, x.tree, x.cache, x.cache, x.n, x.parent),
    "tree_attn_paged": lambda v, x: B.s4c_tree_attn_paged(x.q, x.tree, x.tree, x.pool, x.pool, x.table, x.n, x.parent, S, v.out, 0.0,
                                                          v.attn_status, v.attn_ws),
    "accept_path": lambda v, x: v.accept_path(x.logits, x.parent, x.tokens, B.S4C_GREEDY),
    "accept_path_static": lambda v, x: B.s4c_accept_path_static(x.logits, x.parent, x.tokens, B.S4C_GREEDY, L, v.path, v.accept_len,
                                                                v.accepted_tokens, v.bonus_token),
    "accept_resample": lambda v, x: v.accept_resample(x.logits, x.dp, x.parent, x.tokens, x.u, x.u1),
    "kv_compact": lambda v, x: v.kv_compact(x.tree, x.tree, x.cache, x.cache, x.n),
    "kv_compact_paged": lambda v, x: B.s4c_kv_compact_paged(x.tree, x.tree, x.pool, x.pool, x.table, x.n, v.path, v.accept_len),
    "commit_path": lambda v, x: v.commit_path(x.trees, x.trees, x.caches, x.caches, x.n),
    "commit_path_paged": lambda v, x: B.s4c_commit_path_paged(x.trees, x.trees, x.pools, x.pools, x.table, x.n, v.path, v.accept_len),
    "build_tree": lambda v, x: B.s4c_build_tree(x.logits, x.parent, x.n, 4, x.parent, x.tokens, x.u, x.ws),
    "draft_linear": lambda v, x: B.s4c_draft_linear(x.e, x.e, x.W, x.e, None, x.ws),
    "step": lambda v, x: v.step(x.q, x.tree, x.tree, x.cache, x.cache, x.n, x.parent, x.logits, x.tokens, B.S4C_GREEDY),
}


@pytest.mark.skipif(torch.cuda.is_available(), reason="the stream lookup does not throw where there is a device")
@pytest.mark.filterwarnings("ignore:Accessing the data pointer of FakeTensor")
@pytest.mark.parametrize("name", CALLS)
def test_exceptions_reach_python(name):
    from types import SimpleNamespace
    with FakeTensorMode():
        x = SimpleNamespace(**tensors())
        v = TreeVerifier(Bn, N, H, H, D, S, V, torch.bfloat16, L, S)
        with pytest.raises(RuntimeError, match="No HIP GPUs"):
            CALLS[name](v, x)
