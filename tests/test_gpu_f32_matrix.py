"""GPU parity of both stages on the fp32 matrix instructions (any head width that is a multiple of 16)."""
import numpy as np
import pytest
import torch

from oracle import vista_oracle as O
from paper_2510_22049_amd import binding as V
from paper_2510_22049_amd import inputs as I
from tests.helpers import dev, host64, torch_dtype

pytestmark = pytest.mark.gpu
LENS = [300, 0, 1, 37, 64, 0, 513, 15, 16, 17]
# fp32 products and sums over at most a few hundred terms, exponents of scores up to ten: 1e-5 of the
# block's largest value; bf16 adds half an ulp of the value at the store
PATH = 1e-5


def check(got, want, dtype):
    top = np.abs(want).reshape(want.shape[0], -1).max(axis=1)[:, None, None]
    assert np.all(np.isfinite(got))
    assert np.all(np.abs(got - want) <= (2.0 ** -8 if dtype == "bf16" else 0.0) * np.abs(want) + PATH * top)


def draw(seed, dtype):
    g = np.random.default_rng(seed)
    return lambda shape, s=1.0: I.round_to((g.normal(size=shape) * s).astype(np.float32), dtype)


# head widths 16, 32, 48, 64; one and several chunks of input channels; every count of query units
@pytest.mark.parametrize("H,d,S", [(1, 16, 1), (3, 48, 17), (2, 96, 64), (1, 64, 65), (5, 80, 16), (4, 64, 128), (2, 128, 129),
                                   (4, 256, 300), (8, 128, 512)])
@pytest.mark.parametrize("form,dtype,seg,per_user,self_term", [
    ("softmax", "f32", 0, False, False), ("softmax", "f32", 96, True, True),
    ("silu", "f32", 32, False, True), ("silu", "bf16", 0, True, False), ("softmax", "bf16", 64, False, False)])
def test_stage1(H, d, S, form, dtype, seg, per_user, self_term):
    r = draw(S, dtype)
    off = I.offsets_from_lengths(LENS)
    X, Q = r((off[-1], d)), r((len(LENS), S, d) if per_user else (S, d))
    Wk, Wv = r((d, d), d ** -0.5), r((d, d), d ** -0.5)
    out = torch.full((len(LENS), S, d), float("nan"), device="cuda", dtype=torch_dtype(dtype))
    silu = form == "silu"
    ws = V.vista_summarize(dev(X, dtype), torch.from_numpy(off).cuda(), dev(Q, dtype), dev(Wk, dtype), dev(Wv, dtype), out,
                           H=H, segment_items=seg, self_term=self_term, attn=V.VISTA_ATTN_SILU if silu else V.VISTA_ATTN_SOFTMAX)
    torch.cuda.synchronize()
    assert int(ws[:4].view(torch.int32).item()) == 0
    got, want = host64(out), (O.summarize_silu if silu else O.summarize)(X, off, Q, Wk, Wv, H, self_term=self_term)
    check(got, want, dtype)
    assert np.all(got[1] == 0) and np.all(got[5] == 0)


@pytest.mark.parametrize("H,d", [(1, 16), (3, 96), (2, 96), (1, 64)])     # (bf16 at dh = 32: an odd head count, else another path)
@pytest.mark.parametrize("C,S", [(1, 1), (15, 63), (16, 64), (17, 65), (40, 16), (3, 512)])
@pytest.mark.parametrize("dtype,self_term", [("f32", False), ("f32", True), ("bf16", True)])
def test_stage2(H, d, C, S, dtype, self_term):
    r = draw(C * S, dtype)
    T, Y = r((3, C, d)), r((3, S, d))
    out = torch.full(T.shape, float("nan"), device="cuda", dtype=torch_dtype(dtype))
    V.vista_target_attend(dev(T, dtype), dev(Y, dtype), out, H=H, self_term=self_term)
    check(host64(out), O.target_attend(T, Y, H, self_term=self_term), dtype)


def test_element_aligned_pointers_keep_the_plain_path():
    d, H, S, C = 64, 2, 24, 9
    r = draw(5, "f32")
    off = I.offsets_from_lengths(LENS)
    X, Q, Wk, Wv, T = r((off[-1], d)), r((S, d)), r((d, d), d ** -0.5), r((d, d), d ** -0.5), r((len(LENS), C, d))

    def shifted(x):
        flat = torch.empty(x.size + 1, device="cuda")
        flat[1:].copy_(dev(x, "f32").flatten())
        return flat[1:].view(x.shape)

    out, scored = torch.empty((len(LENS), S, d), device="cuda"), torch.empty(T.shape, device="cuda")
    V.vista_summarize(shifted(X), torch.from_numpy(off).cuda(), shifted(Q), shifted(Wk), shifted(Wv), out, H=H)
    want = O.summarize(X, off, Q, Wk, Wv, H)
    check(host64(out), want, "f32")
    V.vista_target_attend(shifted(T), dev(want.astype(np.float32), "f32"), scored, H=H)
    check(host64(scored), O.target_attend(T, want.astype(np.float32), H), "f32")


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("form", [V.VISTA_ATTN_SOFTMAX, V.VISTA_ATTN_SILU])
def test_users_are_isolated(dtype, form):
    """Infinite rows of one user leave the bits of the users that share its tiles unchanged."""
    d, H, S = 64, 1, 20
    r = draw(9, dtype)
    off = I.offsets_from_lengths([40, 7, 90, 3, 200])
    X, Q, Wk, Wv = r((off[-1], d)), r((S, d)), r((d, d), d ** -0.5), r((d, d), d ** -0.5)

    def run():
        out = torch.empty((5, S, d), device="cuda", dtype=torch_dtype(dtype))
        V.vista_summarize(dev(X, dtype), torch.from_numpy(off).cuda(), dev(Q, dtype), dev(Wk, dtype), dev(Wv, dtype), out, H=H,
                          attn=form)
        return host64(out)

    before = run()
    X[off[1]:off[2]] = np.inf
    X[off[3]:off[4], 5] = -np.inf
    after = run()
    for b in (0, 2, 4):
        assert np.array_equal(before[b], after[b])


@pytest.mark.parametrize("H,d,S", [(1, 64, 16), (1, 64, 64), (2, 128, 33), (4, 64, 49), (3, 144, 17)])
@pytest.mark.parametrize("form,dtype", [("softmax", "f32"), ("silu", "f32"), ("softmax", "bf16")])
@pytest.mark.parametrize("lens", [[1], [16], [31], [1024], LENS, [8, 8, 8, 8, 24, 200, 15, 17]])
def test_segments_of_32_items(H, d, S, form, dtype, lens):
    """The smallest calls: eight waves a workgroup, two for the same queries, whose halves of a tile may hold different users,
    none of a user's items or a single one.  An infinite row of one user leaves the others their bits."""
    r = draw(S + len(lens), dtype)
    off, B, silu = I.offsets_from_lengths(lens), len(lens), form == "silu"
    X, Q, Wk, Wv = r((off[-1], d)), r((S, d)), r((d, d), d ** -0.5), r((d, d), d ** -0.5)
    attn = V.VISTA_ATTN_SILU if silu else V.VISTA_ATTN_SOFTMAX

    def call(X):
        out = torch.full((B, S, d), float("nan"), device="cuda", dtype=torch_dtype(dtype))
        V.vista_summarize(dev(X, dtype), torch.from_numpy(off).cuda(), dev(Q, dtype), dev(Wk, dtype), dev(Wv, dtype), out, H=H, segment_items=32, attn=attn)
        return host64(out)

    got = call(X)
    check(got, (O.summarize_silu if silu else O.summarize)(X, off, Q, Wk, Wv, H), dtype)
    if B > 1:
        bad = int(np.argmax(lens))
        X[off[bad]:off[bad + 1]] = np.inf
        after, rest = call(X), np.arange(B) != bad
        assert np.array_equal(after[rest], got[rest])
