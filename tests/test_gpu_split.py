"""GPU parity of the matrix-core path with split operands (bf16 softmax shapes outside the fixed seed
counts): K, V and weights keep 22 bits and a sign as two fp16 terms, a piece in which these leave too little of a row is formed again
in fp32, so what separates a result from the oracle is the rounding of the bf16 output and of fp32 sums."""
import numpy as np
import pytest
import torch

from oracle import vista_oracle as O
from paper_2510_22049_amd import binding as V
from paper_2510_22049_amd import inputs as I
from tests.helpers import dev, host64

pytestmark = pytest.mark.gpu
LENS = [700, 0, 1, 31, 32, 33, 2100, 64, 0, 95, 1029]


def problem(seed, d, S, per_user=False, xscale=1.0, lens=LENS):
    g = np.random.default_rng(seed)
    off = I.offsets_from_lengths(lens)
    r = lambda shape, s=1.0: I.round_to((g.normal(size=shape) * s).astype(np.float32), "bf16")
    return r((off[-1], d), xscale), off, r((len(lens), S, d) if per_user else (S, d)), r((d, d), d ** -0.5), r((d, d), d ** -0.5)


def check(got, want, path_error):
    """Half a bf16 ulp of the value (2^-8 of it) plus the path's own error relative to the block."""
    top = np.abs(want).reshape(want.shape[0], -1).max(axis=1)[:, None, None]
    assert np.all(np.isfinite(got))
    assert np.all(np.abs(got - want) <= 2.0 ** -8 * np.abs(want) + path_error * top)


def run(X, off, Q, Wk, Wv, H, **kw):
    out = torch.full((len(off) - 1,) + Q.shape[-2:], float("nan"), device="cuda", dtype=torch.bfloat16)
    ws = V.vista_summarize(dev(X, "bf16"), torch.from_numpy(off).cuda(), dev(Q, "bf16"), dev(Wk, "bf16"), dev(Wv, "bf16"),
                           out, H=H, **kw)
    torch.cuda.synchronize()
    assert int(ws[:4].view(torch.int32).item()) == 0
    return host64(out)


# one case on each side of every change of block count per wave and waves per head
@pytest.mark.parametrize("d,H,S", [(64, 2, 1), (64, 2, 64), (64, 2, 65), (64, 2, 100), (64, 2, 161), (64, 2, 257), (64, 2, 512),
                                   (128, 4, 16), (128, 4, 33), (128, 4, 127), (128, 4, 129), (128, 4, 255), (128, 4, 300), (128, 4, 511),
                                   (256, 8, 31), (256, 8, 100), (256, 8, 250), (256, 8, 257), (256, 8, 500)])
@pytest.mark.parametrize("seg,per_user,self_term", [(0, False, False), (64, True, True)])
def test_split_matches_oracle(d, H, S, seg, per_user, self_term):
    X, off, Q, Wk, Wv = problem(S, d, S, per_user)
    got = run(X, off, Q, Wk, Wv, H, segment_items=seg, self_term=self_term)
    want = O.summarize(X, off, Q, Wk, Wv, H, self_term=self_term)
    check(got, want, 1e-4)               # remainders of 2^-17, scores up to ten: 1e-4
    assert np.all(got[1] == 0) and np.all(got[8] == 0)


def test_split_running_maximum():
    """Scores of several tens: tiles beyond the norm bound take the running maximum; the keys' 2^-17
    becomes 2^-17 of a score of about 100 in the exponent."""
    X, off, Q, Wk, Wv = problem(3, 128, 100, xscale=12.0, lens=[300, 77, 1500])
    check(run(X, off, Q, Wk, Wv, 4, segment_items=256), O.summarize(X, off, Q, Wk, Wv, 4), 4e-3)


def test_split_shapes_keep_what_the_plain_path_took():
    """An odd element offset of the history, and a workspace of the plain path's size only."""
    d, H, S = 64, 2, 100
    X, off, Q, Wk, Wv = problem(5, d, S)
    want = O.summarize(X, off, Q, Wk, Wv, H)
    flat = torch.empty(X.size + 1, device="cuda", dtype=torch.bfloat16)
    Xo = flat[1:].view(X.shape)
    Xo.copy_(dev(X, "bf16"))
    a = [torch.from_numpy(off).cuda(), dev(Q, "bf16"), dev(Wk, "bf16"), dev(Wv, "bf16")]
    out = torch.full((len(LENS), S, d), float("nan"), device="cuda", dtype=torch.bfloat16)
    V.vista_summarize(Xo, *a, out, H=H)
    check(host64(out), want, 1e-4)
    B, N, seg = len(LENS), int(off[-1]), 256
    G = (N + seg - 1) // seg
    up = lambda n: (n + 255) // 256 * 256
    plain = 256 + up(4 * G) + up((G + B) * S * (d + 2 * H) * 4) + 2 * up(N * d * 4)
    out.fill_(float("nan"))
    V.vista_summarize(dev(X, "bf16"), *a, out, H=H, workspace=torch.empty(plain, dtype=torch.uint8, device="cuda"))
    check(host64(out), want, 1e-4)
    with pytest.raises(V.VistaError):
        V.vista_summarize(dev(X, "bf16"), *a, out, H=H, workspace=torch.empty(plain - 1, dtype=torch.uint8, device="cuda"))


@pytest.mark.parametrize("B", [1, 3, 64, 65, 200])
def test_first_user_of_a_segment(B):
    """Indexing: Q = 0 and W_v = I make every output the mean of its user's rows; users of 0 to 40 rows
    in segments of 32, so a segment's first user lies anywhere (and behind runs of empty users)."""
    g = np.random.default_rng(B)
    lens = g.integers(0, 41, size=B)
    lens[g.random(B) < 0.3] = 0
    lens[-1] = 5
    off, d, S = I.offsets_from_lengths(lens), 64, 5
    X = np.zeros((off[-1], d), np.float32)
    X[:, 0] = np.repeat(np.arange(B), lens)
    eye = np.eye(d, dtype=np.float32)
    got = run(X, off, np.zeros((S, d), np.float32), eye, eye, 2, segment_items=32)
    assert np.array_equal(got[:, :, 0], np.where(lens > 0, np.arange(B), 0)[:, None].repeat(S, 1))


@pytest.mark.parametrize("bad", [[0, 70, 40, 100], [1, 50, 60, 100], [0, 50, 60, 99], [0, -5, 300, 100]])
def test_offsets_are_checked_on_the_device(bad):
    d, S = 128, 64
    out = torch.zeros((3, S, d), device="cuda", dtype=torch.bfloat16)
    z = lambda *s: torch.zeros(s, device="cuda", dtype=torch.bfloat16)
    ws = V.vista_summarize(z(100, d), torch.tensor(bad, device="cuda"), z(S, d), z(d, d), z(d, d), out, H=4)
    torch.cuda.synchronize()
    assert int(ws[:4].view(torch.int32).item()) == V.VISTA_ERR_OFFSETS


def test_split_users_are_isolated():
    """Infinite rows of one user leave the other users' bits unchanged."""
    lens = [40, 7, 90, 3, 200]
    X, off, Q, Wk, Wv = problem(9, 64, 40, lens=lens)
    before = run(X, off, Q, Wk, Wv, 2)
    X[off[1]:off[2]] = np.inf
    X[off[3]:off[4], 5] = -np.inf
    after = run(X, off, Q, Wk, Wv, 2)
    for b in (0, 2, 4):
        assert np.array_equal(before[b], after[b])


@pytest.mark.parametrize("form,d,H,S,n", [(V.VISTA_ATTN_SOFTMAX, 128, 4, 256, 7001), (V.VISTA_ATTN_SILU, 256, 8, 128, 3000),
                                          (V.VISTA_ATTN_QLA, 128, 4, 40, 5000)])
def test_a_workspace_of_the_base_schedule_gets_the_base_schedule(form, d, H, S, n):
    """Where the fitted segments need more, the smaller workspace is still taken, and the call is bit for bit
    the one with the base segment size given."""
    X, off, Q, Wk, Wv = problem(n, d, S, lens=[n - 90, 0, 90])
    desc = V.summarize_desc(3, S, d, H, V.VISTA_BF16, n, attn=form)
    seg = V.vista_summarize_segment_items(desc)
    base = V.vista_summarize_workspace_bytes(V.summarize_desc(3, S, d, H, V.VISTA_BF16, n, attn=form, segment_items=seg))
    assert base < V.vista_summarize_workspace_bytes(desc)
    ws = torch.empty(base, dtype=torch.uint8, device="cuda")
    got = run(X, off, Q, Wk, Wv, H, attn=form, workspace=ws)
    assert np.array_equal(got, run(X, off, Q, Wk, Wv, H, attn=form, segment_items=seg))
    with pytest.raises(V.VistaError):
        run(X, off, Q, Wk, Wv, H, attn=form, workspace=ws[:base - 1])


@pytest.mark.parametrize("form,d,H,S", [(V.VISTA_ATTN_SOFTMAX, 128, 4, 256), (V.VISTA_ATTN_SOFTMAX, 256, 8, 512), (V.VISTA_ATTN_SOFTMAX, 64, 2, 40),
                                        (V.VISTA_ATTN_QLA, 128, 4, 40), (V.VISTA_ATTN_QLA, 256, 8, 64)])
def test_element_aligned_weights_give_the_same_bits(form, d, H, S):
    """Weights that are not 16-byte aligned are read two bytes at a time into the same operands."""
    X, off, Q, Wk, Wv = problem(S, d, S)

    def shifted(w):
        flat = torch.empty(w.size + 1, device="cuda", dtype=torch.bfloat16)
        flat[1:].copy_(dev(w, "bf16").flatten())
        return flat[1:].view(w.shape)

    out = torch.full((len(LENS), S, d), float("nan"), device="cuda", dtype=torch.bfloat16)
    V.vista_summarize(dev(X, "bf16"), torch.from_numpy(off).cuda(), dev(Q, "bf16"), shifted(Wk), shifted(Wv), out, H=H, attn=form)
    assert np.array_equal(host64(out), run(X, off, Q, Wk, Wv, H, attn=form))


def test_split_keeps_the_precision_of_fp32_operands():
    """Two items a user with nearly equal keys and opposite values: an output is a weight difference times
    a value, so an error of a score shows undamped.  Keys and scores are fp32 sums of 64 and 32 rounded
    terms: about sqrt(96) units of 2^-24 of the largest score, half of which reaches the weights' difference."""
    g = np.random.default_rng(11)
    d, H, S, B = 64, 2, 40, 24
    half, r = d // 2, np.arange(B)
    bf = lambda x: I.round_to(np.asarray(x, dtype=np.float32), "bf16")
    a, c = bf(g.normal(size=(B, half)) * 12.5), bf(g.normal(size=(B, half)))
    a2, j = a.copy(), g.integers(0, half, size=B)
    a2[r, j] = (a[r, j].view(np.uint32) + 0x10000).view(np.float32)          # the next bf16 number
    X = np.empty((2 * B, d), np.float32)
    X[0::2], X[1::2] = np.concatenate([a, c], 1), np.concatenate([a2, -c], 1)
    Wk, Wv = np.zeros((d, d), np.float32), np.zeros((d, d), np.float32)
    Wk[:half], Wv[half:] = bf(g.normal(size=(half, d)) * half ** -0.5), bf(g.normal(size=(half, d)) * half ** -0.5)
    Q, off = bf(g.normal(size=(S, d)) * 12.5), np.arange(0, 2 * B + 1, 2)
    keys = (X.astype(np.float64) @ Wk).reshape(-1, H, d // H)
    smax = np.abs(np.einsum("nhe,she->nsh", keys, Q.reshape(S, H, d // H))).max() * (d // H) ** -0.5
    want, got = O.summarize(X, off, Q, Wk, Wv, H), run(X, off, Q, Wk, Wv, H)
    top = np.abs(X.astype(np.float64) @ Wv).reshape(B, -1).max(axis=1)[:, None, None]
    assert np.all(np.abs(got - want) <= 2.0 ** -8 * np.abs(want) + 0.5 * 96 ** 0.5 * 2.0 ** -24 * smax * top)
@pytest.mark.parametrize("d,H", [(64, 2), (128, 4), (256, 8)])
@pytest.mark.parametrize("rows", [(5,), (33,), (69,), (3, 40, 69)])
def test_split_values_and_keys_that_leave_the_bf16_range(d, H, rows):
    """Values that overflow (or that only bf16 cannot hold) and keys at minus infinity behave as in fp32:
    they reach their own channel, a key at minus infinity takes its item out."""
    g = np.random.default_rng(13)
    S, L = 40, 70                                                 # two full tiles and a ragged one
    bf = lambda x: I.round_to(np.asarray(x, dtype=np.float32), "bf16")
    X, Q = bf(g.normal(size=(2 * L, d))), bf(g.normal(size=(S, d)))
    X[:, -3:] = 0.0
    Wk, Wv = bf(g.normal(size=(d, d)) * d ** -0.5), bf(g.normal(size=(d, d)) * d ** -0.5)
    Wk[-3:], Wv[-3:], Wk[:, -1], Q[:, -1] = 0.0, 0.0, 0.0, 1.0
    Wk[-2, -1] = -2.0                                             # 2^127 in channel -2: the last key is minus infinity
    Wv[-1, [0, 7, 31, d - 1]] = 2.0, -2.0, 1.9921875, 2.0 ** -20  # 2^127 in channel -1: inf, -inf, the largest bf16, 2^107
    Wv[-3, 31] = 1.5 * 2.0 ** 119                                 # 1 in channel -3: beyond the largest bf16, within fp32
    off = np.array([0, L, 2 * L])
    clean = O.summarize(X, off, Q, Wk, Wv, H)
    for r in rows:
        X[r, -1], X[r, -3] = 2.0 ** 127, 1.0
    want, dh = O.summarize(X, off, Q, Wk, Wv, H), d // H
    X[17, -2] = 2.0 ** 127                                        # the item leaves the last head
    want[:, :, -dh:] = O.summarize(np.delete(X, 17, axis=0), np.array([0, L - 1, 2 * L - 1]), Q, Wk, Wv, H)[:, :, -dh:]
    out = torch.full((2, S, d), float("nan"), device="cuda", dtype=torch.bfloat16)
    V.vista_summarize(dev(X, "bf16"), torch.from_numpy(off).cuda(), dev(Q, "bf16"), dev(Wk, "bf16"), dev(Wv, "bf16"), out, H=H)
    got = host64(out)
    assert np.all(np.isposinf(got[0, :, 0])) and np.all(np.isneginf(got[0, :, 7]))
    top = np.abs(want).max(axis=1, keepdims=True)                 # per channel: their sizes differ by 2^100
    near = lambda a, b, t: np.abs(a - b) <= 2.0 ** -8 * np.abs(b) + 1e-4 * t
    rest = np.setdiff1d(np.arange(d), [0, 7] if len(rows) == 1 else [0, 7, 31])    # (several overflow the un-normalised sum)
    assert np.all(near(got[0], want[0], top[0])[:, rest])
    assert np.all(near(got[1], clean[1], np.abs(clean).max(axis=1, keepdims=True)[1]))


@pytest.mark.parametrize("bad", [float("inf"), float("-inf"), float("nan")])
@pytest.mark.parametrize("form,d,H,S,self_term", [
    (V.VISTA_ATTN_SOFTMAX, 128, 4, 256, True), (V.VISTA_ATTN_SOFTMAX, 256, 8, 64, False), (V.VISTA_ATTN_SOFTMAX, 64, 2, 40, True),
    (V.VISTA_ATTN_SILU, 128, 4, 64, True), (V.VISTA_ATTN_QLA, 128, 4, 40, True), (V.VISTA_ATTN_QLA, 256, 8, 64, False)])
def test_a_weight_that_is_not_finite_stays_in_its_column(form, d, H, S, self_term, bad):
    """One such entry of W_v reaches one channel; the others keep their bits.  (The split shapes take other
    products for such tiles: fp32 sums in another order, at most the next bf16 number, 2^-7 of the value,
    plus 1e-5 of the block.)"""
    X, off, Q, Wk, Wv = problem(S + d, d, S, lens=[300, 0, 45])
    before = run(X, off, Q, Wk, Wv, H, attn=form, self_term=self_term)
    r, c = d // 2 + 3, d - 14
    Wv[r, c] = bad
    out = torch.zeros((3, S, d), device="cuda", dtype=torch.bfloat16)
    V.vista_summarize(dev(X, "bf16"), torch.from_numpy(off).cuda(), dev(Q, "bf16"), dev(Wk, "bf16"), dev(Wv, "bf16"), out, H=H,
                      attn=form, self_term=self_term)
    got, rest = host64(out), np.delete(np.arange(d), c)
    one_ulp = 2.0 ** -7 * np.abs(before) + 1e-5 * np.abs(before).max(axis=(1, 2), keepdims=True)
    assert np.all(np.abs(got - before)[:, :, rest] <= (one_ulp[:, :, rest] if S == 40 and form == V.VISTA_ATTN_SOFTMAX else 0.0))
    assert not np.any(np.isfinite(got[[0, 2]][:, :, c]))


@pytest.mark.parametrize("form", [V.VISTA_ATTN_SOFTMAX, V.VISTA_ATTN_SILU])
@pytest.mark.parametrize("users", [4, 70])
@pytest.mark.parametrize("records", [1, 3, 8, 9, 16, 20, 32, 33])
def test_an_infinite_record_keeps_to_its_channel(form, users, records):
    """A value beyond fp32 makes one channel of its user infinite in every record count a batch of the merge can end with (in
    four runs of records for few users, in one for many), and leaves the other channels their bits."""
    d, H, S, seg = 128, 4, 64, 64
    X, off, Q, Wk, Wv = problem(records, d, S, lens=[seg * records] + [65] * (users - 1))
    X[:, -1], Wk[-1], Wv[-1] = 0.0, 0.0, 0.0
    Wv[-1, 40] = 2.0
    clean = run(X, off, Q, Wk, Wv, H, attn=form, segment_items=seg)
    run_of = -(-records // 4) if users == 4 else records
    for last in {run_of, records}:                                # the last record of the first run, of the last
        Y = X.copy()
        Y[seg * last - 7, -1] = 2.0 ** 127
        out = torch.zeros((users, S, d), device="cuda", dtype=torch.bfloat16)
        V.vista_summarize(dev(Y, "bf16"), torch.from_numpy(off).cuda(), dev(Q, "bf16"), dev(Wk, "bf16"), dev(Wv, "bf16"), out, H=H,
                          attn=form, segment_items=seg)
        got = host64(out)
        assert np.all(np.isinf(got[0, :, 40])), f"record {last} of {records}"
        got[0, :, 40] = clean[0, :, 40]
        assert np.array_equal(got, clean)


@pytest.mark.parametrize("form,dtype,d,H,S,n", [
    (V.VISTA_ATTN_SOFTMAX, "bf16", 128, 4, 256, 7001), (V.VISTA_ATTN_SILU, "bf16", 256, 8, 128, 3000), (V.VISTA_ATTN_SOFTMAX, "bf16", 64, 2, 40, 5000),
    (V.VISTA_ATTN_QLA, "bf16", 128, 4, 40, 5000), (V.VISTA_ATTN_SOFTMAX, "f32", 64, 1, 16, 1024), (V.VISTA_ATTN_SILU, "f32", 40, 2, 16, 1024)])
def test_the_reported_segment_size_is_the_one_used(form, dtype, d, H, S, n):
    """With that size given the call writes the same workspace, records and all (another size puts them elsewhere)."""
    X, off, Q, Wk, Wv = problem(n, d, S, lens=[n - 90, 0, 90])
    desc = lambda seg: V.summarize_desc(3, S, d, H, V.VISTA_BF16 if dtype == "bf16" else V.VISTA_F32, n, attn=form, segment_items=seg)
    used = V.vista_summarize_call_segment_items(desc(0))
    bytes_ = max(V.vista_summarize_workspace_bytes(desc(0)), V.vista_summarize_workspace_bytes(desc(used)))

    def call(seg):
        ws = torch.zeros(bytes_, dtype=torch.uint8, device="cuda")
        out = torch.empty((3, S, d), device="cuda", dtype=torch.bfloat16 if dtype == "bf16" else torch.float32)
        V.vista_summarize(dev(X, dtype), torch.from_numpy(off).cuda(), dev(Q, dtype), dev(Wk, dtype), dev(Wv, dtype), out, H=H,
                          segment_items=seg, workspace=ws, attn=form)
        return ws, out

    (ws0, out0), (ws1, out1) = call(0), call(used)
    assert torch.equal(ws0, ws1) and torch.equal(out0, out1)
    assert not torch.equal(ws0, call(used + 32)[0])


@pytest.mark.parametrize("dtype,d,H,S", [("f32", 64, 1, 16), ("f32", 96, 2, 200), ("bf16", 48, 1, 40), ("bf16", 64, 2, 40), ("bf16", 128, 4, 256),
                                         ("bf16", 256, 8, 128)])
@pytest.mark.parametrize("rows", [(64, 128), (128, 160), (0, 64), (128, 700)])
@pytest.mark.parametrize("seg", [0, 64])
def test_items_at_minus_infinity_leave_the_softmax(dtype, d, H, S, rows, seg):
    """Whole tiles and whole segments of them, wherever the segment edges lie."""
    g = np.random.default_rng(17)
    L, dh = 700 + 97, d // H
    r = lambda shape, s=1.0: I.round_to((g.normal(size=shape) * s).astype(np.float32), dtype)
    X, Q, Wk, Wv = r((L + 50, d)), r((S, d)), r((d, d), d ** -0.5), r((d, d), d ** -0.5)
    X[:, -1] = Wk[-1] = Wv[-1] = 0.0
    Q[:, ::dh], Wk[-1, ::dh] = 1.0, -16.0                       # 2^127 in the last channel: every head's first key channel is -inf
    X[rows[0]:rows[1], -1] = 2.0 ** 127
    off, gone = np.array([0, L, L + 50]), rows[1] - rows[0]
    out = torch.full((2, S, d), float("nan"), device="cuda", dtype=torch.float32 if dtype == "f32" else torch.bfloat16)
    V.vista_summarize(dev(X, dtype), torch.from_numpy(off).cuda(), dev(Q, dtype), dev(Wk, dtype), dev(Wv, dtype), out, H=H, segment_items=seg)
    want = O.summarize(np.delete(X, slice(*rows), axis=0), np.array([0, L - gone, L + 50 - gone]), Q, Wk, Wv, H)
    # at fixed bf16 operands (S of 64, 128, 256, 512) the path's own tolerance, else that of fp32 sums
    check(host64(out), want, (2e-2 if dtype == "bf16" and S in (128, 256) else 1e-4))


def records(X, Q, Wk, Wv, H, named=True):
    """One user, one segment: every head's rows [H, S, dh] before their bf16 rounding and in fp64, from the
    partial record (registers [4][lane][4], row 8 (i / 4) + i % 4 + 4 (lane / 32), column lane % 32; then [lane][l, m])."""
    (L, d), S = X.shape, Q.shape[0]
    dh, nqb, seg = d // H, (S + 31) // 32, (L + 31) // 32 * 32
    out = torch.empty((1, S, d), device="cuda", dtype=torch.bfloat16)
    ws = V.vista_summarize(dev(X, "bf16"), torch.tensor([0, L], device="cuda"), dev(Q, "bf16"), dev(Wk, "bf16"), dev(Wv, "bf16"), out,
                           H=H, segment_items=seg if named else 0)
    rec = ws[512:512 + H * nqb * 4608].view(torch.float32).cpu().double().numpy().reshape(H, nqb, 1152)
    o = rec[:, :, :1024].reshape(H, nqb, 4, 2, 32, 4).transpose(0, 1, 4, 2, 3, 5).reshape(H, nqb * 32, dh)
    got = o / rec[:, :, 1024::2].reshape(H, nqb, 2, 32)[:, :, 0].reshape(H, nqb * 32, 1)
    heads = lambda m: (m.astype(np.float64)).reshape(-1, H, dh).transpose(1, 0, 2)
    s = heads(Q) @ heads(X.astype(np.float64) @ Wk).transpose(0, 2, 1) * dh ** -0.5
    w = np.exp(s - s.max(axis=2, keepdims=True))
    return got[:, :S], w @ heads(X.astype(np.float64) @ Wv) / w.sum(axis=2, keepdims=True)


def record_error(X, Q, Wk, Wv, H):
    """The largest error of a head's result (2-norm)."""
    got, want = records(X, Q, Wk, Wv, H)
    return (np.linalg.norm(got - want, axis=(1, 2)) / np.linalg.norm(want, axis=(1, 2))).max()


# plain tiles, references of a row's own, fp32 for what fp16 terms do not hold (both ends), and queries beyond them
@pytest.mark.parametrize("x,q,w", [(1, 1, 1), (1, 4, 1), (1, 16, 1), (0.02, 50, 1), (30, 0.03, 1), (1, 1, 0.01), (1e-5, 1, 1), (400, 0.003, 1),
                                   (0.01, 80, 1), (3e4, 1e-3, 1e-3)])
@pytest.mark.parametrize("d,H,S", [(64, 2, 33), (128, 4, 100), (256, 8, 40)])
def test_split_keeps_fp32_precision_at_every_scale(d, H, S, x, q, w):
    """Operands are right to 2^-23 of their size, products and sums in fp32: against scores of a hundred 2^-23 becomes 2^-17 of
    a weight, averaged over the items that share it; 2^-19 covers all of these scales (three bf16 terms: up to 1.8e-6)."""
    g = np.random.default_rng(S)
    r = lambda shape, s: I.round_to((g.normal(size=shape) * s).astype(np.float32), "bf16")
    assert record_error(r((900, d), x), r((S, d), q), r((d, d), w * d ** -0.5), r((d, d), w * d ** -0.5), H) <= 2.0 ** -19


@pytest.mark.parametrize("d,H,S,per_user", [(64, 2, 100, False), (128, 4, 40, True), (256, 8, 300, False)])
@pytest.mark.parametrize("seg", [0, 512])
def test_split_histories_that_change_their_scale(d, H, S, per_user, seg):
    """Users of very different sizes in one segment, and histories that start small and grow, so that a piece leaves the flat
    reference and then fp16 behind, and all-negative rows: every user keeps its own tolerance."""
    lens = [200, 330, 90, 31, 400, 64, 150]
    X, off, Q, Wk, Wv = problem(21, d, S, per_user, lens=lens)
    X[off[1]:off[2]] *= np.linspace(0.25, 8, lens[1])[:, None]
    X[off[2]:off[3]] *= 2.0 ** -17
    X[off[4]:off[5]] += 1.5 * X[off[4]]                            # a common direction: some seeds score below -10 throughout
    X[off[5]] *= 2.0 ** 9
    X[off[6] + 100:] *= 2.0 ** 12
    X = I.round_to(X, "bf16")
    check(run(X, off, Q, Wk, Wv, H, segment_items=seg), O.summarize(X, off, Q, Wk, Wv, H), 4e-3)     # (as for the running maximum)


@pytest.mark.parametrize("d,H,S,limit", [(64, 2, 40, 16384), (64, 2, 256, 275000), (128, 4, 33, 8192), (128, 4, 96, 237500), (128, 4, 250, 59375),
                                           (64, 2, 255, 162500), (128, 4, 95, 125000), (128, 4, 249, 66291), (128, 4, 205, 80992)])
@pytest.mark.parametrize("beyond", [0, 1])
@pytest.mark.parametrize("self_term", [False, True])
def test_both_sides_of_one_head_a_workgroup(d, H, S, limit, beyond, self_term):
    """Up to these many items a split call takes workgroups of one head, beyond of two: ragged users, one without items, and
    the same again in segments of a named size, which keep two heads.  (The longest user by its first eight queries.)"""
    lens = [1, 0, 33, 700, 64]
    lens.insert(3, limit + beyond - sum(lens))
    X, off, Q, Wk, Wv = problem(31, d, S, lens=lens)
    got = run(X, off, Q, Wk, Wv, H, self_term=self_term)
    assert np.all(got[1] == 0)
    few = [0, 2, 4, 5]
    Xs = np.concatenate([X[off[b]:off[b + 1]] for b in few])
    check(got[few], O.summarize(Xs, I.offsets_from_lengths([lens[b] for b in few]), Q, Wk, Wv, H, self_term=self_term), 1e-4)
    check(got[3:4, :8], O.summarize(X[off[3]:off[4]], np.array([0, lens[3]]), Q[:8], Wk, Wv, H, self_term=self_term), 1e-4)
    named = run(X, off, Q, Wk, Wv, H, self_term=self_term, segment_items=2048)
    top = np.abs(got).reshape(6, -1).max(axis=1)[:, None, None]
    assert np.all(np.abs(got - named) <= 2.0 ** -7 * np.abs(got) + 1e-5 * top)      # at most the next bf16 number


@pytest.mark.parametrize("d,H", [(64, 2), (128, 4), (256, 8)])
@pytest.mark.parametrize("seg", [0, 256])
def test_split_queries_of_zeros_beside_values_that_fp16_does_not_hold(d, H, seg):
    """No score leaves any bound, whatever the keys: values and keys that fp16 does not hold are seen all the same."""
    X, off, Q, Wk, Wv = problem(41, d, 40, lens=[300, 128])
    X[70:75] *= 2.0 ** 20
    Q[:] = 0.0
    check(run(X, off, Q, Wk, Wv, H, segment_items=seg), O.summarize(X, off, Q, Wk, Wv, H), 1e-4)


def row_errors(X, Q, Wk, Wv, H, named):
    got, want = records(X, Q, Wk, Wv, H, named)
    return np.linalg.norm(got - want, axis=2) / np.linalg.norm(want, axis=2)


@pytest.mark.parametrize("d,H,S", [(64, 2, 33), (128, 4, 100), (128, 4, 300), (256, 8, 40), (256, 8, 257)])
@pytest.mark.parametrize("score", [2.0, 10.4, 15.0, 18.2, 19.4, 30.0, 50.0, 100.0])
@pytest.mark.parametrize("L,spread,named", [(99, 0.0, False), (99, 0.05, True), (3000, 0.0, True), (3000, 0.3, True)])
def test_split_weights_far_below_a_row_s_best_count(d, H, S, score, L, spread, named):
    """A history that begins with a row of zeros (score 0, value 0) and goes on with items that score 2^-score: they alone make
    the result, row by row.  fp32 sums: 2^-19 where keys have 22 bits and a sign, and 2^-22 of the score in the exponent, the same for
    all items of a row."""
    g = np.random.default_rng(S)
    bf = lambda x: I.round_to(np.asarray(x, dtype=np.float32), "bf16")
    Wk, Wv = np.zeros((d, d), np.float32), bf(np.abs(g.normal(size=(d, d))) * d ** -0.5)
    Wk[0], Wv[0] = 1.0, 0.0                                      # channel 0 makes the keys, the others the values
    X = bf(np.abs(g.normal(size=(L, d))))
    X[:, 0] = bf(score / (32 ** 0.5 * 1.4427) * (1 + spread * g.normal(size=L) / score))
    X[0] = 0.0
    Q = bf(-1.0 - g.integers(0, 2, size=(S, 1)) / 64 + np.zeros((S, d)))
    assert row_errors(X, Q, Wk, Wv, H, named).max() <= 2.0 ** -19 + score * 2.0 ** -22


@pytest.mark.parametrize("d,H,S", [(64, 2, 33), (128, 4, 100), (256, 8, 300)])
@pytest.mark.parametrize("k,q,x", [(1000, 3e-4, 1), (3000, 1e-4, 1), (4000, 1e-5, 1), (1, 3e-4, 60), (1, 1e-6, 1), (1e-6, 1e6, 1), (1e4, 3e-6, 30)])
@pytest.mark.parametrize("named", [True, False])
def test_split_small_queries_meet_large_keys(d, H, S, k, q, x, named):
    """Scores of ordinary size from operands that are not: as at every scale, and in rows."""
    g = np.random.default_rng(S)
    r = lambda shape, s: I.round_to((g.normal(size=shape) * s).astype(np.float32), "bf16")
    X, Q, Wk, Wv = r((128, d), x), r((S, d), q), r((d, d), k * d ** -0.5), r((d, d), d ** -0.5)
    Q[1] *= 2.0 ** -10                                            # and a row of much smaller ones among them
    assert row_errors(X, Q, Wk, Wv, H, named).max() <= 2.0 ** -18.5     # (a row instead of all rows of a head)


@pytest.mark.parametrize("d,H,S", [(64, 2, 100), (128, 4, 33), (256, 8, 40)])
@pytest.mark.parametrize("small", [8, 12, 16, 24, 40])
@pytest.mark.parametrize("L,named", [(100, False), (800, True)])
def test_split_a_small_value_among_large_ones(d, H, S, small, L, named):
    """The item that all of the weight goes to has values 2^-small of the others', whose part of the result is 2^-60: the result is known
    as any other, to 2^-20 where two fp16 terms are cut off below and to fp32 sums of d products, some 2^-21."""
    g = np.random.default_rng(S)
    bf = lambda x: I.round_to(np.asarray(x, dtype=np.float32), "bf16")
    Wk, Wv = np.zeros((d, d), np.float32), bf(g.normal(size=(d, d)) * d ** -0.5)
    Wk[0], Wv[0] = 1.0, 0.0
    X = bf(g.normal(size=(L, d)))
    X[:, 0] = -13.0
    X[70, 1:] *= 2.0 ** -small
    X[70, 0] = 0.0
    assert row_errors(X, bf(np.ones((S, d))), Wk, Wv, H, named).max() <= 2.0 ** -19


@pytest.mark.parametrize("d,H,S", [(64, 2, 33), (64, 2, 100), (128, 4, 100), (256, 8, 300)])
@pytest.mark.parametrize("seg", [0, 64, 2048])
def test_split_users_whose_own_queries_differ_in_scale(d, H, S, seg):
    """Pieces of one tile and of many, each user's queries of another size over items of the inverse: a unit for each piece, formed
    two tiles ahead.  (Scores as at unit scale: 1e-4 of the block.)"""
    lens = [1, 40, 700, 0, 31, 32, 33, 5, 64, 300, 2, 95]
    X, off, Q, Wk, Wv = problem(S, d, S, per_user=True, lens=lens)
    for b, e in enumerate([0, 9, -9, 3, -14, 14, 0, -7, 30, -30, 5, 11]):
        Q[b] *= 2.0 ** e
        X[off[b]:off[b + 1]] *= 2.0 ** -e
    check(run(X, off, Q, Wk, Wv, H, segment_items=seg), O.summarize(X, off, Q, Wk, Wv, H), 1e-4)


@pytest.mark.parametrize("d,H,S", [(64, 2, 40), (128, 4, 100), (256, 8, 100)])
@pytest.mark.parametrize("times", [2.0 ** 12, 2.0 ** 90, float("inf")])
def test_split_a_user_s_own_queries_beyond_fp16(d, H, S, times):
    """Large queries of one user, over small keys, are his alone: the others keep their bits."""
    lens = [40, 300, 90, 3, 200]
    X, off, Q, Wk, Wv = problem(17, d, S, per_user=True, lens=lens)
    before = run(X, off, Q, Wk, Wv, H)
    with np.errstate(invalid="ignore"):
        Q[1] = Q[1] * times
    if np.isfinite(times):
        X[off[1]:off[2]] *= 2.0 ** -12
    out = torch.full((5, S, d), float("nan"), device="cuda", dtype=torch.bfloat16)
    V.vista_summarize(dev(X, "bf16"), torch.from_numpy(off).cuda(), dev(Q, "bf16"), dev(Wk, "bf16"), dev(Wv, "bf16"), out, H=H)
    got = host64(out)
    for b in (0, 2, 3, 4):
        assert np.array_equal(before[b], got[b])
    if times == 2.0 ** 12:
        check(got[1:2], O.summarize(X[off[1]:off[2]], np.array([0, lens[1]]), Q[1:2], Wk, Wv, H), 1e-4)
    elif times == 2.0 ** 90:                                       # every weight goes to the best item
        check(got[1:2], O.summarize(X[off[1]:off[2]], np.array([0, lens[1]]), Q[1:2], Wk, Wv, H), 1e-4)
