"""Attention whose keys are divided between workgroups, on sequences much shorter than max_cache_len, empty or of an
invalid length, with a workspace that holds another call's numbers: against the oracle, through s4c_tree_attn (contiguous
and paged) and through the step's own merge.  tests/test_attn_division.py checks that the cases are divided as they say."""
from dataclasses import dataclass
from typing import Tuple

import numpy as np
import pytest
import torch

from oracle import s4c_oracle as O
from paper_2506_14158_amd import binding as B, synth
from paper_2506_14158_amd.verify import TreeVerifier
from tests.util import attn_errors, np_to_torch

# Rows that see one or a few keys are nearly rows of V, with values up to 4: their own rounding to the storage type (half
# an ulp is 2^-9 of the value in bf16, 2^-12 in fp16, up to twice that within a binade) comes on top of the error of the sums,
# so the absolute bar grows with the value.  (floor, share of the value), and the relative error of a row.
TOL = {"f32": (1e-5, 0.0, 1e-5), "bf16": (5e-3, 2.0 ** -8, 2e-2), "f16": (1.25e-3, 2.0 ** -11, 2.5e-3)}


@dataclass(frozen=True)
class Case:
    name: str
    kind: str                      # "split": equal runs per unit; "balanced": equal shares of all units
    B: int
    Hkv: int
    G: int
    D: int
    N: int
    dtype: str
    max_len: int
    lens: Tuple[int, ...]          # repeated over the batch; beyond max_len or negative: flagged


CASES = [
    # one key tile: an empty prefix, a flagged length; one more: a prefix of one row, of a whole tile; several
    Case("rows256", "split", 8, 8, 4, 128, 64, "bf16", 8192, (0, 8193, -1, 64, 1, 300, 65, 0)),
    Case("rows256-d64", "split", 3, 8, 4, 64, 37, "bf16", 2049, (0, 2050, 70)),
    Case("rows128", "split", 2, 4, 8, 128, 16, "f16", 9000, (0, 129)),
    Case("rows64", "split", 2, 8, 1, 128, 60, "bf16", 5000, (4, 5001)),
    Case("rows32", "split", 3, 4, 1, 128, 30, "bf16", 5000, (0, 5001, 33)),
    Case("rows32-f32", "split", 2, 4, 2, 64, 15, "f32", 3000, (0, 40)),
    # fewer key tiles than teams: teams without a share; then enough of them, shares that end inside units; both kinds of rows
    Case("shares-rows256", "balanced", 13, 8, 4, 128, 47, "f16", 5003, (1, 64, 17, 30)),
    Case("shares-rows256-mixed", "balanced", 13, 8, 4, 128, 47, "bf16", 5003, (5, 900, 0, 64, 5004, 129)),
    Case("shares-rows64", "balanced", 3, 32, 1, 128, 37, "bf16", 24000, (64, 33, 1)),
    Case("shares-rows64-mixed", "balanced", 3, 32, 1, 128, 37, "f16", 24000, (700, 0, 40)),
    Case("rows32-d64", "split", 5, 18, 1, 64, 20, "bf16", 3000, (32, 0, 1, 500, -1)),
    Case("shares-rows32", "balanced", 13, 16, 1, 64, 20, "bf16", 3000, (32, 0, 1, 500, -1)),
    Case("shares-f32", "balanced", 3, 30, 2, 64, 40, "f32", 3000, (2, 50, 333)),
    # long shares of few rows: the key groups of a workgroup see different maxima
    Case("shares-rows32-long", "balanced", 13, 16, 2, 64, 1, "f16", 3000, (3000, 2901)),
    Case("shares-rows32-long-bf16", "balanced", 13, 16, 1, 64, 32, "bf16", 3000, (2777, 3000, 1500)),
    Case("shares-rows32-long-f32", "balanced", 7, 20, 2, 64, 13, "f32", 2500, (2500, 2431)),
    Case("shares-rows32-deep", "balanced", 33, 8, 1, 128, 20, "bf16", 7960, (500, 0, 33, 7961, 64)),   # four key groups
    Case("70-sequences", "split", 70, 2, 1, 64, 20, "bf16", 3000, (1, 0, 64, 100, 31)),
    Case("shares-70-sequences", "balanced", 70, 3, 1, 64, 20, "bf16", 3000, (1, 0, 64, 100, 31)),
]


def plan_inputs(c):
    """B, Hkv, N, M, max_cache_len, then rows, keys and workgroups per CU of the kernel's tile for the case, whether it is 16-bit
    data of head size 128, and CUs"""
    M = c.N * c.G
    wide = c.dtype != "f32" and c.D == 128
    if c.dtype != "f32" and M > 64:
        tile = (128, 64, 2 if c.D == 64 else 1) if M <= 128 else (256, 64, 1)
    elif M <= 32 and (c.D == 64 or (wide and c.max_len >= 4096 and c.B * c.Hkv * c.max_len >= 7168 * 256)):
        tile = (32, 32, 2 if c.D == 64 and c.dtype != "f32" else 1)
    else:
        tile = (64, 32, 1 if c.dtype == "f32" and c.D == 128 else 2)
    return (c.B, c.Hkv, c.N, M, c.max_len) + tile + (int(wide), 256)


def inputs(c):
    lens = np.array([c.lens[b % len(c.lens)] for b in range(c.B)], dtype=np.int32)
    top = int(lens[lens <= c.max_len].max(initial=1))
    cfg = synth.scaled(synth.CONFIGS[4], name=c.name, B=c.B, Hq=c.Hkv * c.G, Hkv=c.Hkv, D=c.D, N=c.N, dtype=c.dtype, P=top, V=500,
                       levels=min(c.N, 6), widths=(8, 4, 3, 2, 2, 2, 2, 2), index=0)
    par, at = synth.make_parent(cfg), synth.make_attn_inputs(cfg)
    ref, st = O.tree_attn(at.q, at.k_tree, at.v_tree, at.k_cache, at.v_cache, lens, par)     # (beyond the capacity: flagged, zeros)
    return cfg, par, at, lens, ref, st


def check(c, got, status, ref, st):
    assert np.array_equal(status.cpu().numpy(), st)
    assert torch.isfinite(got.float()).all()
    amax, rel = attn_errors(got, ref)
    floor, share, row = TOL[c.dtype]
    excess = float((np.abs(got.float().cpu().numpy().astype(np.float64) - ref) - share * np.abs(ref)).max())
    assert excess <= floor and rel <= row, (c.name, amax, rel, excess)


@pytest.mark.gpu
@pytest.mark.parametrize("case", CASES, ids=lambda c: c.name)
def test_short_sequences_of_a_divided_launch(case):
    cfg, par, at, lens, ref, st = inputs(case)
    dev = {k: np_to_torch(getattr(at, k)) for k in ("q", "k_tree", "v_tree", "k_cache", "v_cache")}
    n, parent = torch.from_numpy(lens).cuda(), torch.from_numpy(par).cuda()
    S_cap = case.max_len + case.N
    big = lambda x: torch.full((case.B, case.Hkv, S_cap, case.D), float("nan"), dtype=x.dtype, device="cuda")
    kc, vc = big(dev["k_cache"]), big(dev["v_cache"])                                        # nothing beyond the lengths is read
    kc[:, :, :cfg.S_cap], vc[:, :, :cfg.S_cap] = dev["k_cache"], dev["v_cache"]
    tv = TreeVerifier(case.B, case.N, cfg.Hq, case.Hkv, case.D, S_cap, cfg.V, dev["q"].dtype, cfg.levels, case.max_len)
    args = (dev["q"], dev["k_tree"], dev["v_tree"])
    tv.attn_ws.fill_(0x7E)                                                                   # 8e37 as floats
    tv.tree_attn(*args, kc, vc, n, parent)
    check(case, tv.out, tv.attn_status, ref, st)

    page = 64
    blocks = -(-S_cap // page)
    order = torch.randperm(case.B * blocks, device="cuda").view(case.B, blocks)
    table = order.to(torch.int32)
    pool = lambda x: torch.zeros(case.B * blocks, case.Hkv, page, case.D, dtype=x.dtype, device="cuda")
    kp, vp = pool(kc), pool(vc)
    for b in range(case.B):
        for p in range(-(-cfg.S_cap // page)):
            m = min(page, S_cap - p * page)
            kp[order[b, p], :, :m], vp[order[b, p], :, :m] = kc[b, :, p * page:p * page + m], vc[b, :, p * page:p * page + m]
    tv.attn_ws.fill_(0x7E)
    out = torch.full_like(tv.out, float("nan"))
    # (the same plan as above: max_cache_len decides, not the capacity)
    B.s4c_tree_attn_paged(*args, kp, vp, table, n, parent, case.max_len, out, 0.0, tv.attn_status, tv.attn_ws)
    check(case, out, tv.attn_status, ref, st)

    tv.attn_ws.fill_(0x7E)
    tv.out.fill_(float("nan"))
    logits = torch.randn(case.B, case.N, cfg.V, device="cuda").to(dev["q"].dtype)
    tv.step(*args, kc, vc, n.clone(), parent, logits, torch.zeros(case.B, case.N, dtype=torch.int32, device="cuda"), B.S4C_GREEDY)
    check(case, tv.out, tv.attn_status, ref, st)
