"""Test plumbing shared by the GPU parity tests (no arithmetic of the method)."""
import numpy as np
import torch

from paper_2510_22049_amd import binding as V

TOL = {"f32": 1e-4, "bf16": 2e-2}     # max error per output block relative to the block's max |value|


def torch_dtype(name):
    return torch.float32 if name == "f32" else torch.bfloat16


def dev(x: np.ndarray, dtype: str) -> torch.Tensor:
    """Storage-rounded fp32 host values -> device tensor of the storage dtype (exact)."""
    return torch.from_numpy(np.ascontiguousarray(x)).to("cuda").to(torch_dtype(dtype))


def host64(t: torch.Tensor) -> np.ndarray:
    return t.detach().to(torch.float32).cpu().numpy().astype(np.float64)


def block_errors(got: np.ndarray, want: np.ndarray) -> np.ndarray:
    """max |got - want| / max |want| over each leading-index block (one user)."""
    g = got.reshape(got.shape[0], -1)
    w = want.reshape(want.shape[0], -1)
    den = np.abs(w).max(axis=1)
    den = np.where(den == 0, 1.0, den)
    return np.abs(g - w).max(axis=1) / den


def floored_errors(got: np.ndarray, want: np.ndarray, floor: float = 1e-3) -> np.ndarray:
    """Element-wise |got - want| / max(|want|, floor x the block's max |want|), worst element per block.
    Reported as information only: near-zero, sign-changing outputs make a bare element-wise ratio
    meaningless, the floor keeps it finite."""
    g = got.reshape(got.shape[0], -1)
    w = want.reshape(want.shape[0], -1)
    top = np.abs(w).max(axis=1, keepdims=True)
    den = np.maximum(np.abs(w), floor * np.where(top == 0, 1.0, top))
    return (np.abs(g - w) / den).max(axis=1)


def assert_blocks_close(got, want, dtype, what=""):
    assert np.all(np.isfinite(got)), f"{what}: non-finite output"
    err = block_errors(got, want)
    worst = int(err.argmax())
    assert err[worst] <= TOL[dtype], f"{what}: block {worst} error {err[worst]:.3e} > {TOL[dtype]:.0e}"
    return float(err.max())


def assert_in_value_hull(out: torch.Tensor, values: torch.Tensor, what="", slack=2.0 ** -7):
    """Property that holds at any size: softmax weights are non-negative and sum to one, so every
    output channel of a block lies between the smallest and the largest value of that channel
    (out [..., rows, d] against values [..., n, d], compared on the device in fp32; `slack` x the
    channel's largest magnitude allows for the bf16 roundings of values, weights and output)."""
    v = values.float()
    lo, hi = v.amin(dim=-2, keepdim=True), v.amax(dim=-2, keepdim=True)
    tol = slack * torch.maximum(lo.abs(), hi.abs())
    o = out.float()
    assert bool(((o >= lo - tol) & (o <= hi + tol)).all()), f"{what}: output outside the hull of its values"


def short_history_limit(form, d, S):
    """Largest history, users beyond the first counted as items, that the bf16 matrix-core kernels of S = 64, 128, 256, 512
    give to workgroups of half the heads (tests/test_schedule_host.py pins it against the library)."""
    if d == 256:
        return 8192 if S == 64 else {"softmax": 32768, "silu": 20480}[form] if S == 512 else {"softmax": 16384, "silu": 12288}[form]
    if form == "silu" and S == 128:
        return 65536
    return {64: 131072, 128: 131072, 256: 229376, 512: 98304}[S]


def user_as_items(form, d, S, own_queries=False):
    if d == 256:
        return 2048 if S == 64 else 384 if form == "silu" else 192 if S < 512 else 3072 if own_queries else 2048
    if form == "silu":
        return (768 if own_queries else 320) if S == 128 else 128
    return (1024 if own_queries else 768) if S == 512 else 640 if own_queries else 384


def always_short(d, S):
    return 12288 if d == 128 else 4096 if S < 256 else 6144


def is_short_history(form, d, S, N, B, own_queries=False, limit=None):
    limit = short_history_limit(form, d, S) if limit is None else limit
    return N <= always_short(d, S) or N + user_as_items(form, d, S, own_queries) * (B - 1) <= limit


def takes_one_head(form, d, S, N, B, own_queries=False):
    """The shortest of these go to workgroups of one head, where the call leaves the segment size open."""
    if (d == 256 and S < 256) or not is_short_history(form, d, S, N, B, own_queries, short_history_limit(form, d, S) // 8 * 7):
        return False
    if d == 256 or S == 512:
        return True
    few = 16384 if S == 64 else {"softmax": 49152, "silu": 53248}[form] if S == 128 else {"softmax": 57344, "silu": 40960}[form]
    return N <= few * (0.4 + 0.6 * 32.0 / (B + 31.0))


def fitted_segment(form, d, S, N, B, own_queries=False):
    """Segment size of those kernels before any limit of the workspace (histories of up to 131 072 items)."""
    whole = 4 if d == 256 else 2 if S == 512 else 1                  # groups of heads
    share = lambda groups: -(-(-(-N // (256 // groups))) // 32) * 32
    if takes_one_head(form, d, S, N, B, own_queries):
        return max(128, share(8 if d == 256 else 4))
    if not is_short_history(form, d, S, N, B, own_queries):
        return max(128, share(whole))
    by_root = (int(1.5 * N ** 0.5) + 16) // 32 * 32 if d == 128 and S < 512 else 0
    return max(128, share(2 * whole), by_root)


def workgroups_taken(form, off, d, H, S, own_queries=False, segment_items=0):
    """Which kind of workgroup a call of those kernels takes, as the library's rules put it: at the fitted segment size as
    above (named, halves in place of one head), at another one (named, or the base schedule's where the workspace has a limit) by
    the number of workgroups."""
    B, N = len(off) - 1, int(off[-1])
    desc = V.summarize_desc(B, S, d, H, V.VISTA_BF16, N, own_queries, segment_items=segment_items,
                            attn=V.VISTA_ATTN_SILU if form == "silu" else V.VISTA_ATTN_SOFTMAX)
    seg = V.vista_summarize_call_segment_items(desc)
    if seg == fitted_segment(form, d, S, N, B, own_queries):
        if takes_one_head(form, d, S, N, B, own_queries):
            return "half" if segment_items else "one"
        return "half" if is_short_history(form, d, S, N, B, own_queries) else "whole"
    few = N + 128 * B <= short_history_limit(form, d, S)
    halves = -(-N // seg) * (8 if d == 256 else 4 if S == 512 else 2)
    half = few or halves <= 256 if d == 128 else halves <= 288 if few else halves <= 256 and S != 64
    return "half" if half else "whole"


def takes_half_workgroups(form, off, d, H, S, own_queries=False, segment_items=0):
    return workgroups_taken(form, off, d, H, S, own_queries, segment_items) == "half"
