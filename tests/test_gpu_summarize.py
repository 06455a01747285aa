"""GPU parity of the MFMA stage-1 path (bf16, head width 32) against the CPU oracle."""
import numpy as np
import pytest
import torch

from oracle import vista_oracle as O
from paper_2510_22049_amd import binding as V
from paper_2510_22049_amd import inputs as I
from tests.helpers import (assert_blocks_close, block_errors, dev, host64, is_short_history, short_history_limit, takes_half_workgroups, user_as_items,
                           workgroups_taken)

pytestmark = pytest.mark.gpu


def bf(x):
    return I.round_to(np.asarray(x, dtype=np.float32), "bf16")


def run(X, off, Q, Wk, Wv, H, **kw):
    B = len(off) - 1
    S, d = Q.shape[-2:]
    out = torch.full((B, S, d), float("nan"), device="cuda", dtype=torch.bfloat16)
    offd = torch.from_numpy(np.asarray(off, dtype=np.int64)).cuda()
    ws = V.vista_summarize(dev(X, "bf16"), offd, dev(Q, "bf16"), dev(Wk, "bf16"), dev(Wv, "bf16"), out, H=H, **kw)
    torch.cuda.synchronize()
    assert int(ws[:4].view(torch.int32).item()) == 0
    return host64(out)


def problem(seed, lens, d, S, per_user=False, xscale=1.0):
    g = np.random.default_rng(seed)
    off = I.offsets_from_lengths(lens)
    X = bf(g.normal(size=(off[-1], d)) * xscale)
    Q = bf(g.normal(size=(len(lens), S, d) if per_user else (S, d)))
    Wk, Wv = bf(g.normal(size=(d, d)) / np.sqrt(d)), bf(g.normal(size=(d, d)) / np.sqrt(d))
    return X, off, Q, Wk, Wv


LENS = [700, 0, 1, 31, 32, 33, 2100, 64, 0, 95, 1029]


@pytest.mark.parametrize("d,H,S", [(128, 4, 256), (128, 4, 64), (128, 4, 128), (128, 4, 512), (256, 8, 512), (256, 8, 256),
                                   (256, 8, 128), (256, 8, 64)])
@pytest.mark.parametrize("seg", [0, 64, 992])
def test_mfma_jagged_matches_oracle(d, H, S, seg):
    """Empty, single-item, one-tile, ragged and multi-segment users; shared queries."""
    X, off, Q, Wk, Wv = problem(1, LENS, d, S)
    got = run(X, off, Q, Wk, Wv, H, segment_items=seg)
    want = O.summarize(X, off, Q, Wk, Wv, H)
    assert_blocks_close(got, want, "bf16", f"d={d} S={S} seg={seg}")
    assert np.all(got[1] == 0) and np.all(got[8] == 0)


@pytest.mark.parametrize("lens,seg,half", [(LENS, 64, True), ([5000], 128, True), ([9000, 33, 0, 120000, 1, 64, 20031, 150000], 2048, False)])
def test_both_orders_of_a_tile_agree(lens, seg, half):
    """S = 256 at d = 128 takes a tile in one order of instructions for shared queries and in another for queries of the
    users' own (launch_for_shape; were both sent to one kernel, this would compare it with itself): the same sums, so the
    same bits where every user's own are the shared ones."""
    X, off, Q, Wk, Wv = problem(9, lens, 128, 256)
    own = np.repeat(Q[None], len(lens), axis=0)
    for per_user in (False, True):
        assert takes_half_workgroups("softmax", off, 128, 4, 256, per_user, seg) == half
    shared = run(X, off, Q, Wk, Wv, 4, segment_items=seg)
    assert np.array_equal(shared, run(X, off, own, Wk, Wv, 4, segment_items=seg))
    few = [b for b in range(len(lens)) if lens[b] <= 9000]
    want = O.summarize(np.concatenate([X[off[b]:off[b + 1]] for b in few]), I.offsets_from_lengths([lens[b] for b in few]), Q, Wk, Wv, 4)
    assert_blocks_close(shared[few], want, "bf16", f"ordered tile, seg={seg}")


@pytest.mark.parametrize("lens,seg", [([700, 0, 1, 31, 2100, 64, 95, 1029], 64), ([9000, 33, 120000, 20031, 0, 1], 2048)])
@pytest.mark.parametrize("per_user", [False, True])
def test_the_ordered_tile_of_512_seeds_agrees_with_the_free_one(lens, seg, per_user):
    """S = 512 at d = 128 takes the ordered tile for queries of either kind, in waves that project and waves that only attend.  Its
    waves hold the seeds that those of two calls of S = 256 with queries of the users' own do (the free tile, launch_for_shape), and up
    to eight users both merge in four runs: the same bits."""
    X, off, Q, Wk, Wv = problem(10, lens, 128, 512, per_user)
    own = Q if per_user else np.repeat(Q[None], len(lens), axis=0)
    got = run(X, off, Q, Wk, Wv, 4, segment_items=seg)
    for half in (slice(0, 256), slice(256, 512)):
        assert np.array_equal(got[:, half], run(X, off, own[:, half], Wk, Wv, 4, segment_items=seg))


@pytest.mark.parametrize("d,H,S", [(128, 4, 256), (256, 8, 512)])
def test_mfma_per_user_queries(d, H, S):
    X, off, Q, Wk, Wv = problem(2, LENS, d, S, per_user=True)
    got = run(X, off, Q, Wk, Wv, H, segment_items=512, offsets_host=torch.from_numpy(off))
    assert_blocks_close(got, O.summarize(X, off, Q, Wk, Wv, H), "bf16", "per-user queries")


@pytest.mark.parametrize("d,H,S", [(128, 4, 256), (256, 8, 512)])
@pytest.mark.parametrize("scale", [0.03, 0.5])
def test_mfma_scale_override(d, H, S, scale):
    """A non-default score scale reaches the kernel (it is folded into the key weights)."""
    X, off, Q, Wk, Wv = problem(8, [700, 0, 33, 1300], d, S)
    got = run(X, off, Q, Wk, Wv, H, segment_items=256, scale=scale)
    want = O.summarize(X, off, Q, Wk, Wv, H, scale=scale)
    assert_blocks_close(got, want, "bf16", f"scale={scale}")
    assert block_errors(O.summarize(X, off, Q, Wk, Wv, H)[[0, 3]], want[[0, 3]]).max() > 5e-2   # the override matters


def test_mfma_large_scores_mix_both_softmax_routes():
    """Item norms straddle the bound |q||k| <= 60 (base 2): tiles switch from the constant
    reference to the running maximum inside a piece."""
    X, off, Q, Wk, Wv = problem(3, [300, 77, 1500], 128, 256, xscale=6.0)
    X[40:60] = bf(X[40:60] / 6.0)               # a stretch of small items inside a large-score user
    got = run(X, off, Q, Wk, Wv, 4, segment_items=256)
    assert_blocks_close(got, O.summarize(X, off, Q, Wk, Wv, 4), "bf16", "xscale=6")


def test_mfma_running_maximum_route_everywhere():
    """Huge key norms in channels the queries do not look at: every tile fails the norm bound
    (so the running-maximum route runs throughout) while the scores themselves stay moderate."""
    g = np.random.default_rng(31)
    d, S = 128, 256
    lens = [257, 40, 900]
    off = I.offsets_from_lengths(lens)
    X = g.normal(size=(off[-1], d))
    Q = g.normal(size=(S, d))
    for h in range(4):
        X[:, 32 * h + 16:32 * h + 32] *= 300.0
        Q[:, 32 * h + 16:32 * h + 32] = 0.0
    X[:, ::7] -= 3.0                            # shift the scores so their maximum is far from 0
    X, Q = bf(X), bf(Q)
    eye = np.eye(d, dtype=np.float32)
    Wv = bf(g.normal(size=(d, d)) / np.sqrt(d) / 50)
    got = run(X, off, Q, eye, Wv, 4, segment_items=128)
    assert_blocks_close(got, O.summarize(X, off, Q, eye, Wv, 4), "bf16", "all-general")


def test_mfma_all_scores_very_negative():
    """Every score sits near -260 (base 2) through a constant channel pair: a reference
    maximum stuck at 0 would underflow every weight to 0/0; the shift itself cancels exactly."""
    X, off, Q, Wk, Wv = problem(4, [200, 45, 1000], 128, 64)
    eye = np.eye(128, dtype=np.float32)
    for h in range(4):
        X[:, 32 * h] = 32.0
        Q[:, 32 * h] = -32.0
    got = run(X, off, Q, eye, Wv, 4, segment_items=128)
    assert_blocks_close(got, O.summarize(X, off, Q, eye, Wv, 4), "bf16", "negative scores")


@pytest.mark.parametrize("big,seg", [(11.0, 64), (11.0, 0), (16.0, 96)])
def test_mfma_beacon_rows_are_found_exactly(big, seg):
    """Indexing, bit-exact: query i is made to select one row of the user (first, last, tile
    edges, middle); the output must be that row's integer payload, exactly."""
    d, H, S = 128, 4, 64
    lens = [1, 2, 31, 32, 33, 64, 65, 0, 700, 1503, 97]
    off = I.offsets_from_lengths(lens)
    g = np.random.default_rng(5)
    X = bf(g.normal(size=(off[-1], d)))
    X[:, :32] = 0
    X[:, 16:32] = g.integers(0, 200, size=(off[-1], 16))          # payload of ordinary rows
    Q = np.zeros((S, d), np.float32)
    want = {}
    for b, L in enumerate(lens):
        picks = [p for p in (0, L - 1, 31, 32, 63, L // 2) if 0 <= p < L]
        for i, pos in enumerate((0, L - 1, 31, 32, 63, L // 2)):
            if not 0 <= pos < L:
                continue
            row = off[b] + pos
            X[row, i] = big
            X[row, 16:19] = (b + 1, pos % 256, pos // 256)
            want[(b, i)] = (b + 1, pos % 256, pos // 256)
    for i in range(6):
        Q[i, i] = big
    eye = np.eye(d, dtype=np.float32)
    got = run(X, off, bf(Q), eye, eye, H, segment_items=seg)
    for (b, i), code in want.items():
        L = lens[b]
        rows = off[b] + np.array([p for p in (0, L - 1, 31, 32, 63, L // 2) if 0 <= p < L])
        same = [r for r in rows if X[r, i] == big]
        if len(same) > 1:
            continue                                              # query i has two beacons in a tiny user
        found = got[b, i, 16:19]            # weights of the other rows are < 2^-30: far below half a unit
        assert tuple(np.rint(found)) == code and np.abs(found - code).max() < 1e-4, (b, i, found, code)


def test_mfma_is_bitwise_reproducible_and_isolated():
    """Same inputs -> same bits; poisoning one user's rows leaves the others' bits unchanged."""
    X, off, Q, Wk, Wv = problem(6, [500, 260, 1200, 33], 128, 256)
    a = run(X, off, Q, Wk, Wv, 4, segment_items=256)
    for _ in range(5):
        assert np.array_equal(a, run(X, off, Q, Wk, Wv, 4, segment_items=256))
    X2 = X.copy()
    X2[off[1]:off[2]] = bf(X2[off[1]:off[2]] * 3 + 1)
    c = run(X2, off, Q, Wk, Wv, 4, segment_items=256)
    for u in (0, 2, 3):
        assert np.array_equal(a[u], c[u])
    assert not np.array_equal(a[1], c[1])


def test_mfma_agrees_with_plain_path_on_gpu():
    """Cross-check (not the oracle): the fp32 matrix kernels on the same bf16-representable inputs."""
    X, off, Q, Wk, Wv = problem(7, [400, 90, 0, 800], 128, 256)
    got = run(X, off, Q, Wk, Wv, 4)
    out32 = torch.empty((4, 256, 128), device="cuda")
    V.vista_summarize(dev(X, "f32"), torch.from_numpy(off).cuda(), dev(Q, "f32"), dev(Wk, "f32"), dev(Wv, "f32"),
                      out32, H=4)
    torch.cuda.synchronize()
    assert block_errors(got, host64(out32)).max() < 2e-2


@pytest.mark.parametrize("d,H,S", [(128, 4, 256), (128, 4, 128), (64, 1, 16)])
def test_degenerate_batches(d, H, S):
    """No items at all (every user empty), and a batch whose only content is one item."""
    g = np.random.default_rng(21)
    Q = bf(g.normal(size=(S, d)))
    Wk, Wv = bf(g.normal(size=(d, d)) / np.sqrt(d)), bf(g.normal(size=(d, d)) / np.sqrt(d))
    got = run(np.zeros((0, d), np.float32), [0, 0, 0, 0], Q, Wk, Wv, H)
    assert got.shape == (3, S, d) and np.all(got == 0)
    X = bf(g.normal(size=(1, d)))
    got = run(X, [0, 0, 1, 1], Q, Wk, Wv, H)
    want = O.summarize(X, [0, 0, 1, 1], Q, Wk, Wv, H)
    assert np.all(got[0] == 0) and np.all(got[2] == 0)
    assert_blocks_close(got[1:2], want[1:2], "bf16", "one item")
    assert np.all(got[1] == got[1][0])          # a single item: every query returns its value row


def test_nothing_is_written_outside_out_and_the_stated_workspace():
    """Canary bytes before and after `out` and after the workspace's stated size survive the call
    (jagged users, several segments, both kernel families)."""
    for d, H, S, dtype in ((128, 4, 256, "bf16"), (64, 2, 24, "f32")):
        g = np.random.default_rng(71)
        lens = [700, 0, 33, 1300]
        off = I.offsets_from_lengths(lens)
        r = lambda shape, s=1.0: I.round_to((g.normal(size=shape) * s).astype(np.float32), dtype)
        X, Q, Wk, Wv = r((off[-1], d)), r((S, d)), r((d, d), d ** -0.5), r((d, d), d ** -0.5)
        tdt = torch.bfloat16 if dtype == "bf16" else torch.float32
        esz = 2 if dtype == "bf16" else 4
        pad = 4096
        n_out = len(lens) * S * d * esz
        raw = torch.full((pad + n_out + pad,), 0xA5, dtype=torch.uint8, device="cuda")
        out = raw[pad:pad + n_out].view(tdt).view(len(lens), S, d)
        desc = V.summarize_desc(len(lens), S, d, H, V.VISTA_BF16 if dtype == "bf16" else V.VISTA_F32, int(off[-1]),
                                segment_items=128)
        need = V.vista_summarize_workspace_bytes(desc)
        wraw = torch.full((need + pad,), 0x5A, dtype=torch.uint8, device="cuda")
        V.vista_summarize(dev(X, dtype), torch.from_numpy(off).cuda(), dev(Q, dtype), dev(Wk, dtype), dev(Wv, dtype), out,
                          H=H, segment_items=128, workspace=wraw[:need], offsets_host=torch.from_numpy(off))
        torch.cuda.synchronize()
        assert bool((raw[:pad] == 0xA5).all()) and bool((raw[pad + n_out:] == 0xA5).all()), "write outside out"
        assert bool((wraw[need:] == 0x5A).all()), "write beyond the stated workspace size"
        assert_blocks_close(host64(out), O.summarize(X, off, Q, Wk, Wv, H), dtype, "canary case")


BLOCKS = [(512, 0), (512, 1), (512, 2), (512, 3), (512, 4), (512, 9), (512, 10), (512, 15), (256, 2), (128, 3), (64, 1)]


@pytest.mark.parametrize("S,block,longest", [(S, b, 2047) for S, b in BLOCKS] +
                         [(S, b, 27000 if S == 512 else 17000) for S, b in BLOCKS if (S, b) not in ((512, 0), (512, 2))])
def test_queries_of_one_block_beyond_the_bound(S, block, longest):
    """d = 256: the waves of a head hold unequal shares of the queries (at S = 512 in workgroups of half the heads, and from
    24 576 items with a thousand or more a user in whole ones); the wave whose block leaves the score bound takes the
    running maximum, the others do not, and every query gets its own result."""
    lens = [900, 1, 33, longest]
    assert is_short_history("softmax", 256, S, sum(lens), 4) == (longest == 2047) and (S != 512 or longest == 2047 or sum(lens) >= 24576)
    X, off, Q, Wk, Wv = problem(40 + block, lens, 256, S)
    Q[32 * block:32 * block + 32] *= 5.0          # exact in bf16 up to its rounding; |q| |k| passes 60, scores stay near 20
    Q = bf(Q)
    want = O.summarize(X, off, Q, Wk, Wv, 8)
    for seg in (960,) if longest == 2047 else (960, 0):
        assert_blocks_close(run(X, off, Q, Wk, Wv, 8, segment_items=seg), want, "bf16", f"S={S} block={block} seg={seg}")


@pytest.mark.parametrize("per_user,users", [(False, 24), (False, 25), (True, 16), (True, 17)])
def test_both_sides_of_the_uneven_query_split(per_user, users):
    """d = 256, S = 512, whole workgroups: 24 576 items (65 536 with queries of their own) of 1024 (4096) a user take the
    uneven split, a user more the even one."""
    items = 65536 if per_user else 24576
    lens = [700, 0, 33] + [items // users] * (users - 3)
    lens[0] += items - sum(lens)
    assert not is_short_history("softmax", 256, 512, items, users, per_user)
    X, off, Q, Wk, Wv = problem(61, lens, 256, 512, per_user=per_user)
    got = run(X, off, Q, Wk, Wv, 8)
    for b in (0, 1, 2, 3, users - 1):              # the longest, the one without items, the shortest and two ordinary ones
        s = slice(off[b], off[b + 1])
        want = O.summarize(X[s], [0, off[b + 1] - off[b]], Q[b] if per_user else Q, Wk, Wv, 8)
        assert_blocks_close(got[b:b + 1], want, "bf16", f"user {b}")
    assert np.all(np.isfinite(got)) and np.all(got[1] == 0)


LIMITS = [("softmax", 128, 4, 64, 240), ("softmax", 128, 4, 128, 240), ("softmax", 128, 4, 256, 200), ("softmax", 128, 4, 512, 80),
          ("silu", 128, 4, 64, 300), ("silu", 128, 4, 128, 80), ("silu", 128, 4, 256, 200), ("silu", 128, 4, 512, 100),
          ("softmax", 256, 8, 64, 2), ("softmax", 256, 8, 128, 20), ("softmax", 256, 8, 256, 20), ("softmax", 256, 8, 512, 5),
          ("silu", 256, 8, 64, 2), ("silu", 256, 8, 128, 10), ("silu", 256, 8, 256, 10), ("silu", 256, 8, 512, 10)]


@pytest.mark.parametrize("form,d,H,S,users", LIMITS)
@pytest.mark.parametrize("beyond", [0, 1])
def test_both_sides_of_the_short_history_limit(form, d, H, S, users, beyond):
    """A history at the limit, users counted as items, goes to workgroups of half the heads, one item more to whole ones:
    ragged users, one without items, tiles and segments that end inside them, default and short segments."""
    lens = ([1, 0, 33, 2011] + [40] * users)[:users - 1]
    items = short_history_limit(form, d, S) - user_as_items(form, d, S) * (users - 1) + beyond
    lens.insert(2, items - sum(lens))
    X, off, Q, Wk, Wv = problem(50, lens, d, S)
    assert takes_half_workgroups(form, off, d, H, S) == (not beyond)
    silu = form == "silu"
    want = (O.summarize_silu if silu else O.summarize)(X, off, Q, Wk, Wv, H)
    for seg in (0, 480):
        got = run(X, off, Q, Wk, Wv, H, segment_items=seg, attn=V.VISTA_ATTN_SILU if silu else V.VISTA_ATTN_SOFTMAX)
        assert_blocks_close(got, want, "bf16", f"{form} d={d} S={S} N={items} seg={seg}")
        assert all(np.all(got[b] == 0) for b in range(users) if lens[b] == 0)


EDGES = ["self", "own", "mixed", "negative", "infinite weight", "aligned to an element", "codec"]


@pytest.mark.parametrize("form,edge", [("softmax", e) for e in EDGES] + [("silu", e) for e in EDGES if e != "negative"])
@pytest.mark.parametrize("d,H,S", [(128, 4, 64), (128, 4, 128), (128, 4, 256), (128, 4, 512), (256, 8, 64), (256, 8, 128), (256, 8, 256), (256, 8, 512)])
def test_whole_workgroups_on_the_edges(form, d, H, S, edge):
    """The same users alone (workgroups of half the heads) and in front of one so long that workgroups are whole: same
    segments, so the same records in the same order.  Bits are equal, but at d = 256, S = 512, where a wave holds other
    queries and the running maximum starts at other tiles; and right by the oracle.  The edges: the self term and a
    scale, queries of their own, scores on both sides of the bound (SiLU: several hundred either way), all of them near
    -260, a weight that is not finite, weights at element alignment, the fused codec."""
    lens = [700, 0, 1, 31, 32, 33, 1100, 64, 0, 95, 1029] + [9, 0, 4] * (20 if d == 128 else 14)
    silu, B = form == "silu", len(lens)
    X, off, Q, Wk, Wv = problem(90 + S, lens, d, S, per_user=edge == "own")
    long = short_history_limit(form, d, S)
    X, off = np.concatenate([X, np.resize(X, (long, d))]), np.append(off, off[-1] + long)
    Q = np.concatenate([Q, Q[:1]]) if edge == "own" else Q
    if edge == "mixed" and silu:
        Q = bf(Q * 12)
    elif edge == "mixed":
        X = bf(X * 6)
        X[40:60] = bf(X[40:60] / 6)
    elif edge == "negative":
        Wk = np.eye(d, dtype=np.float32)
        X[:, ::32], Q[..., ::32] = 32.0, -32.0
    elif edge == "infinite weight":
        Wv[d // 2 + 3, d - 14] = np.inf

    def call(users):
        o = off[:users + 1]
        assert takes_half_workgroups(form, o, d, H, S, edge == "own", 128) == (users == B)
        q = dev(Q[:users] if edge == "own" else Q, "bf16")
        w = [dev(m, "bf16") for m in (Wk, Wv)]
        if edge == "aligned to an element":
            flat = [torch.empty(d * d + 1, device="cuda", dtype=torch.bfloat16) for _ in w]
            for f, m in zip(flat, w):
                f[1:].copy_(m.flatten())
            w = [f[1:].view(d, d) for f in flat]
        args = (dev(X[:o[-1]], "bf16"), torch.from_numpy(o).cuda(), q, *w)
        kw = dict(H=H, attn=V.VISTA_ATTN_SILU if silu else V.VISTA_ATTN_SOFTMAX, self_term=edge == "self", scale=0.2 if edge == "self" else 0.0,
                  segment_items=128)
        if edge == "codec":
            codes, scales = torch.full((users, S, d), 99, device="cuda", dtype=torch.int8), torch.zeros((users, S, H), device="cuda")
            V.vista_summarize_q8(*args, codes, scales, **kw)
            return O.dequantize_summaries(codes.cpu().numpy()[:B], scales.cpu().numpy()[:B])
        out = torch.full((users, S, d), float("nan"), device="cuda", dtype=torch.bfloat16)
        V.vista_summarize(*args, out, **kw)
        return host64(out)[:B]

    assert B * H * (S // 32) > 512                 # both calls merge a user's records in one run
    alone, among = call(B), call(B + 1)
    if (d, S) != (256, 512):
        assert np.array_equal(alone, among, equal_nan=True)
    if edge == "infinite weight":
        rest = np.delete(np.arange(d), d - 14)
        assert np.all(np.isfinite(among[:, :, rest])) and not np.any(np.isfinite(among[[0, 6]][:, :, d - 14]))
        Wv[d // 2 + 3, d - 14], among = 0.0, among[:, :, rest]
    want = (O.summarize_silu if silu else O.summarize)(X[:off[B]], off[:B + 1], Q[:B] if edge == "own" else Q, Wk, Wv, H,
                                                       **(dict(self_term=True, scale=0.2) if edge == "self" else {}))
    if edge == "infinite weight":
        want = want[:, :, rest]
    if edge == "codec":     # on top of the path's 2e-2 half a step of the codec, 1/254 of a group's largest computed magnitude
        assert np.all(np.abs(among - want) <= (2e-2 + 1 / 254) * np.abs(want).max(axis=(1, 2), keepdims=True) * 1.02)
    else:
        # mixed: keys six times as long.  Their bf16 rounding moves a score by 2^-9 / sqrt(3) x 6 = 0.007 (one sigma), 0.03 at the worst of
        # the 10^6 there are; between two items of equal weight and opposite value that is 0.25 x 0.03 x 2 of the largest value
        slack = 0.015 if edge == "mixed" and not silu else 0.0
        assert np.all(np.isfinite(among)) and block_errors(among, want).max() <= 2e-2 + slack, f"{form} d={d} S={S} {edge}"


@pytest.mark.parametrize("form,d,H,S", [(f, *s) for f in ("softmax", "silu") for s in ((128, 4, 64), (128, 4, 128), (128, 4, 256), (128, 4, 512),
                                                                                          (256, 8, 256), (256, 8, 512))])
@pytest.mark.parametrize("edge", ["shared", "own", "self", "mixed"])
def test_workgroups_of_one_head(form, d, H, S, edge):
    """Short histories whose segment size is left open take one head a workgroup, a named size halves: both right by the
    oracle, and where no score leaves the bound (or the form has none) the same bits in segments of the same size.  Ragged users, runs
    of empty ones, a single item, users that end on tiles and segments."""
    lens = [1, 0, 0, 33, 128, 700, 31, 1027, 64, 95] + [9, 0, 4] * 5
    silu = form == "silu"
    X, off, Q, Wk, Wv = problem(70 + S, lens, d, S, per_user=edge == "own")
    if edge == "mixed":
        X[40:300] = bf(X[40:300] * 4.8)    # |q| |k| up to 68 on both sides of 60; bf16 keys cost 2^-9 of a score, up to 0.017 of the block here
    attn = V.VISTA_ATTN_SILU if silu else V.VISTA_ATTN_SOFTMAX
    kw = dict(attn=attn, self_term=edge == "self")
    fitted = V.vista_summarize_call_segment_items(V.summarize_desc(len(lens), S, d, H, V.VISTA_BF16, int(off[-1]), edge == "own", attn=attn,
                                                                   self_term=edge == "self"))
    assert workgroups_taken(form, off, d, H, S, edge == "own") == "one" and workgroups_taken(form, off, d, H, S, edge == "own", fitted) == "half"
    got, halves = run(X, off, Q, Wk, Wv, H, **kw), run(X, off, Q, Wk, Wv, H, segment_items=fitted, **kw)
    want = (O.summarize_silu if silu else O.summarize)(X, off, Q, Wk, Wv, H, self_term=edge == "self")
    assert_blocks_close(got, want, "bf16", f"one head, {form} d={d} S={S} {edge}")
    assert_blocks_close(halves, want, "bf16", f"halves, {form} d={d} S={S} {edge}")
    assert all(np.all(got[b] == 0) for b in range(len(lens)) if lens[b] == 0)
    if silu or edge != "mixed":
        assert np.array_equal(got, halves)
    elif S > 64:                           # half the blocks a wave: a bound on scores of other queries, which is left at other tiles
        assert not np.array_equal(got, halves)
