"""The cases whose speed this framework is judged by: one pass each through the public entry points.

Shapes are those of `paper_2510_22049_amd/inputs.py`'s five workloads and of the ranges around
them: head width 32 in bf16 (64 in the small fp32 configuration), 16 to 512 seeds, histories from
a few hundred to a million items, jagged batches, candidate lists from a handful to thousands.

    listed()          the cases by name
    draw(rng)         one more case of the same ranges
    prepare(case, s)  what a program holds before the call: inputs (from the seed alone), offsets,
                      weights, output buffers and the workspace
    run(state)        one pass
    work(case)        bytes and flops the pass cannot do without
    tolerance(case)   how far another correct implementation at the same precision may differ
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2510_22049_amd import binding as V

FORMS = {"softmax": V.VISTA_ATTN_SOFTMAX, "silu": V.VISTA_ATTN_SILU, "qla": V.VISTA_ATTN_QLA}
DTYPES = {"bf16": torch.bfloat16, "f32": torch.float32}


# ------------------------------------------------------------------------------- the cases

def _stage1(path, form, users, items, d, H, S, dtype="bf16", spread=1.0, self_term=False, host_offsets=True,
            per_user=False):
    return {"path": path, "form": form, "users": users, "items": items, "spread": spread, "d": d, "H": H, "S": S,
            "dtype": dtype, "self_term": self_term, "host_offsets": host_offsets, "per_user": per_user}


def _stage2(path, users, C, d, H, S, self_term=False):
    return {"path": path, "users": users, "C": C, "d": d, "H": H, "S": S, "dtype": "bf16", "self_term": self_term}


def _two_stage(users, items, C, d, H, S):
    return {"path": "two_stage", "users": users, "items": items, "spread": 0.5, "C": C, "d": d, "H": H, "S": S,
            "dtype": "f32"}


def _stack(users, items, C, d, H, S):
    return {"path": "stack", "users": users, "items": items, "spread": 0.5, "C": C, "d": d, "H": H, "S": S,
            "dtype": "bf16"}


def listed():
    return [
        # the tiny configuration: fp32, one head of 64; a unit-test or notebook call, all latency
        {"name": "tiny_fp32", **_two_stage(1, 1024, 32, 64, 1, 16)},
        # one user came back: the summaries of a single ordinary history are renewed online, the
        # offsets exist on the device only
        {"name": "refresh_one_user", **_stage1("summarize", "softmax", 1, 7001, 128, 4, 256, host_offsets=False)},
        # the jagged batch: 64 users, lognormal lengths around 8k (the headline workload)
        {"name": "jagged", **_stage1("summarize", "softmax", 64, 768597, 128, 4, 256)},
        # a narrower model with a seed count that is no power of two
        {"name": "odd_seeds", **_stage1("summarize", "softmax", 48, 300007, 64, 2, 100)},
        # lifelong histories: 8 users of a million items (split over the chip and merged)
        {"name": "lifelong", **_stage1("summarize", "softmax", 8, 8_000_000, 128, 4, 256, spread=0.0)},
        # the whole path: two stacked layers with the gated block between, then candidate attention
        {"name": "end_to_end", **_stack(256, 14_026_438, 256, 256, 8, 512)},
        # SiLU score form, 128 seeds that also attend to themselves
        {"name": "silu_self", **_stage1("summarize", "silu", 64, 500_003, 128, 4, 128, self_term=True)},
        # quasi-linear attention over the jagged batch
        {"name": "qla", **_stage1("summarize", "qla", 64, 768597, 128, 4, 256)},
        # its gradients: the training direction
        {"name": "qla_backward", **_stage1("backward", "qla", 64, 768597, 128, 4, 256)},
        # serving: 1024 users, 512 candidates each, over cached summaries
        {"name": "serving", **_stage2("attend", 1024, 512, 128, 4, 256)},
        # the int8 cache: summaries are written through the codec and scored from it, ragged sizes
        {"name": "serving_int8", **_stage2("cache", 300, 333, 128, 4, 128, self_term=True)},
        # two requests with short candidate lists: latency again
        {"name": "serving_small", **_stage2("attend", 2, 100, 128, 4, 256)},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    path = rng.choice(["summarize", "summarize", "summarize", "odd", "silu", "qla", "backward", "attend", "cache",
                       "two_stage", "stack"])
    d, H = rng.choice([(128, 4), (128, 4), (256, 8)])
    S = rng.choice([64, 128, 256, 512])
    self_term = rng.random() < 0.25
    host = rng.random() < 0.75
    if path == "two_stage":
        H = rng.choice([1, 2, 4])
        return _two_stage(_log(rng, 1, 8), _log(rng, 300, 8000), _log(rng, 8, 128), 64, H, _log(rng, 16, 64))
    if path == "odd":
        d, H = rng.choice([(64, 2), (128, 4), (256, 8)])
        return _stage1("summarize", "softmax", _log(rng, 1, 64), _log(rng, 3000, 300_007), d, H,
                       rng.randint(16, 512), self_term=self_term, host_offsets=host)
    if path in ("summarize", "silu"):
        return _stage1("summarize", "silu" if path == "silu" else "softmax", _log(rng, 1, 128),
                       _log(rng, 2000, 3_000_000), d, H, S, spread=rng.choice([0.0, 0.5, 1.0]), self_term=self_term,
                       host_offsets=host, per_user=rng.random() < 0.2)
    if path == "qla":
        return _stage1("summarize", "qla", _log(rng, 1, 128), _log(rng, 2000, 3_000_000), d, H, rng.randint(16, 512),
                       self_term=self_term, host_offsets=host)
    if path == "backward":
        users = _log(rng, 1, 128)
        return _stage1("backward", "qla", users, min(1_500_000, users * _log(rng, 500, 20_000)), d, H,
                       rng.randint(16, 512), self_term=self_term, host_offsets=host)
    if path == "stack":
        return _stack(_log(rng, 2, 64), _log(rng, 20_000, 2_000_000), _log(rng, 16, 512), d, H, S)
    # multiples of 32 up to 256, of 64 beyond: what stage 1 writes and the serving side caches
    S = rng.choice([32 * rng.randint(1, 8), 64 * rng.randint(5, 8)])
    users = _log(rng, 1, 1024)
    C = _log(rng, 8, min(4096, max(9, 600_000 // users)))
    return _stage2(path, users, C, d, H, S, self_term=self_term)


# ------------------------------------------------------------------------------- a pass

def _lengths(case, seed):
    """Lengths of the users' histories: lognormal shares of exactly `items` rows."""
    g = np.random.default_rng(seed)
    share = np.exp(case["spread"] * g.standard_normal(case["users"]))
    cut = np.floor(np.cumsum(share) / share.sum() * case["items"]).astype(np.int64)
    cut[-1] = case["items"]
    return np.concatenate([np.zeros(1, dtype=np.int64), cut])


def prepare(case, seed):
    dt = DTYPES[case["dtype"]]
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    B, d, H, S = case["users"], case["d"], case["H"], case["S"]

    def normal(*shape, std=1.0):
        t = torch.empty(shape, device="cuda", dtype=dt).normal_(generator=g)
        return t.mul_(std) if std != 1.0 else t

    def empty(*shape, dtype=dt):
        return torch.empty(shape, device="cuda", dtype=dtype)

    st = {"case": case, "H": H}
    path = case["path"]
    if path in ("summarize", "backward", "two_stage", "stack"):
        N = case["items"]
        off = torch.from_numpy(_lengths(case, seed))
        st["off"] = off.cuda()
        st["off_host"] = off if case.get("host_offsets", True) else None
        st["X"] = normal(N, d)
        st["Q"] = normal(B, S, d) if case.get("per_user") else normal(S, d)
        st["Wk"], st["Wv"] = normal(d, d, std=d ** -0.5), normal(d, d, std=d ** -0.5)
        st["summ"] = empty(B, S, d)
        form = FORMS[case.get("form", "softmax")]
        self_term = case.get("self_term", False)
        code = V.VISTA_BF16 if dt == torch.bfloat16 else V.VISTA_F32
        desc = V.summarize_desc(B, S, d, H, code, N, per_user_q=bool(case.get("per_user")) or path == "stack",
                                attn=form, self_term=self_term)
        if path == "backward":
            st["dO"] = normal(B, S, d)
            st["dQ"], st["dK"], st["dV"] = empty(B, S, d), empty(N, d), empty(N, d)
            st["dKs"], st["dVs"] = (empty(B, S, d), empty(B, S, d)) if self_term else (None, None)
            bytes_ = V.lib().vista_qla_backward_workspace_bytes(desc)
        else:
            bytes_ = V.vista_summarize_workspace_bytes(desc)
        st["ws"] = torch.empty(max(bytes_, 256), device="cuda", dtype=torch.uint8)
    if path == "stack":
        F = 2 * d
        st["Wk2"], st["Wv2"] = normal(d, d, std=d ** -0.5), normal(d, d, std=d ** -0.5)
        st["Wg"], st["Wu"], st["Wo"] = normal(d, F, std=d ** -0.5), normal(d, F, std=d ** -0.5), normal(F, d, std=F ** -0.5)
        st["q2"], st["summ2"] = empty(B, S, d), empty(B, S, d)
    if path in ("attend", "cache"):
        st["summ"] = normal(B, S, d)
    if path == "cache":
        st["codes"], st["scales"] = empty(B, S, d, dtype=torch.int8), empty(B, S, H, dtype=torch.float32)
    if "C" in case:
        st["cand"] = normal(B, case["C"], d)
        st["scored"] = empty(B, case["C"], d)
    return st


def run(st):
    case, H = st["case"], st["H"]
    path = case["path"]
    if path == "summarize":
        V.vista_summarize(st["X"], st["off"], st["Q"], st["Wk"], st["Wv"], st["summ"], H=H,
                          offsets_host=st["off_host"], workspace=st["ws"], attn=FORMS[case["form"]],
                          self_term=case["self_term"])
        return st["summ"]
    if path == "backward":
        V.vista_qla_backward(st["X"], st["off"], st["Q"], st["Wk"], st["Wv"], st["dO"], st["dQ"], st["dK"], st["dV"],
                             H=H, offsets_host=st["off_host"], workspace=st["ws"], d_self_keys=st["dKs"],
                             d_self_values=st["dVs"])
        grads = {"dQ": st["dQ"], "dK": st["dK"], "dV": st["dV"]}
        if case["self_term"]:
            grads.update(dKs=st["dKs"], dVs=st["dVs"])
        return grads
    if path == "two_stage":
        V.vista_summarize(st["X"], st["off"], st["Q"], st["Wk"], st["Wv"], st["summ"], H=H,
                          offsets_host=st["off_host"], workspace=st["ws"])
        V.vista_target_attend(st["cand"], st["summ"], st["scored"], H=H)
        return {"summaries": st["summ"], "scored": st["scored"]}
    if path == "stack":
        V.vista_summarize(st["X"], st["off"], st["Q"], st["Wk"], st["Wv"], st["summ"], H=H,
                          offsets_host=st["off_host"], workspace=st["ws"])
        V.vista_sglu_ffn(st["summ"], st["Wg"], st["Wu"], st["Wo"], st["q2"])
        V.vista_summarize(st["X"], st["off"], st["q2"], st["Wk2"], st["Wv2"], st["summ2"], H=H,
                          offsets_host=st["off_host"], workspace=st["ws"])
        V.vista_target_attend(st["cand"], st["summ2"], st["scored"], H=H)
        return {"layer1": st["summ"], "queries2": st["q2"], "layer2": st["summ2"], "scored": st["scored"]}
    if path == "attend":
        V.vista_target_attend(st["cand"], st["summ"], st["scored"], H=H, self_term=case["self_term"])
        return st["scored"]
    V.vista_quantize_summaries(st["summ"], st["codes"], st["scales"], H=H)
    V.vista_target_attend_q8(st["cand"], st["codes"], st["scales"], st["scored"], H=H, self_term=case["self_term"])
    return {"codes": st["codes"], "scales": st["scales"], "scored": st["scored"]}


# ------------------------------------------------------------------------------- its price

def work(case):
    """Every input read once, every output written once; multiply-adds of the definitions."""
    path, d, H, S, B = case["path"], case["d"], case["H"], case["S"], case["users"]
    e = 2 if case["dtype"] == "bf16" else 4
    C = case.get("C", 0)
    N = case.get("items", 0)
    dh = d // H
    attend = {"bytes": e * B * d * (2 * C + S), "flops": 4 * B * C * S * d}
    if path == "attend":
        return attend
    if path == "cache":      # bf16 summaries in, codes and scales out, candidates in, results out
        return {"bytes": e * B * d * (2 * C + S) + B * S * (d + 4 * H), "flops": attend["flops"]}
    queries = B * S if case.get("per_user") else S
    if case.get("form") == "qla":
        fwd = {"bytes": e * (N * d + queries * d + 2 * d * d + B * S * d),
               "flops": N * (4 * d * d + 2 * d * dh) + 2 * B * S * d * dh}
        if path == "summarize":
            return fwd
        return {"bytes": e * (3 * N * d + queries * d + 2 * d * d + 2 * B * S * d + (2 * B * S * d if case["self_term"] else 0)),
                "flops": N * (4 * d * d + 6 * d * dh) + 4 * B * S * d * dh}
    layer = {"bytes": e * (N * d + queries * d + 2 * d * d + B * S * d), "flops": N * (4 * d * d + 4 * S * d)}
    if path == "summarize":
        return layer
    if path == "two_stage":  # the summaries are an output as well as stage 2's input
        return {"bytes": layer["bytes"] + 2 * e * B * C * d, "flops": layer["flops"] + attend["flops"]}
    # two layers over one history (a history that outgrows the caches is read twice), the gated block of
    # inner width 2d, the candidates
    F = 2 * d
    return {"bytes": e * (2 * N * d + S * d + 4 * d * d + 3 * d * F + 3 * B * S * d + 2 * B * C * d),
            "flops": 2 * layer["flops"] + 6 * B * S * d * F + attend["flops"]}


def tolerance(case):
    """About four times the error against the same expressions in fp64, measured on every listed case
    and fourteen drawn ones (2-norm of the difference over 2-norm of the fp64 result)."""
    if case["dtype"] == "f32":
        return {"rel": 2e-6}             # fp32 sums: 2.4e-7 to 3.0e-7
    if case["path"] == "backward":
        # The gradients carry SiLU'(Z) of a state that sums a user's L items: where an entry of Z is near
        # zero the derivative moves with Z's absolute error, which grows like sqrt(L).  Measured
        # 2.6e-4 sqrt(L) for dK and dV (2.8e-2 at L = 12k, 1.3e-2 at L = 2.9k), 2.4e-3 for dQ; twice
        # that, because the operands' own roundings, which cause it, are the same in any bf16 version.
        return {"rel": max(1e-2, 5.2e-4 * math.sqrt(case["items"] / case["users"]))}
    if case["path"] == "stack":
        return {"rel": 1.5e-2}           # four bf16 stages in a row: up to 4.6e-3
    if case["path"] == "cache":
        return {"rel": 1e-2, "differ": 0.0}   # the codec works in fp32 on both sides: codes are equal
    return {"rel": 1e-2}                 # bf16 operands, fp32 sums: 1.7e-3 to 3.2e-3
