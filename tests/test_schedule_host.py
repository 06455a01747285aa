"""Host-only checks of the split-L schedule (integer work, bit-exact): the tile walk of the streaming
kernels, reported by vista_summarize_schedule, against a brute-force statement of the same schedule at
the base segment size and at the one a call uses."""
import numpy as np
import pytest

from paper_2510_22049_amd import binding as V
from paper_2510_22049_amd import inputs as I
from tests.helpers import always_short, fitted_segment, is_short_history, short_history_limit, takes_one_head, user_as_items


def desc(B, N, seg=0, S=256, d=128, H=4):
    return V.summarize_desc(B, S, d, H, V.VISTA_BF16, N, segment_items=seg)


def brute_force_tiles(off, seg):
    """Segments of `seg` flat rows, cut at user boundaries, each piece cut into tiles of 32."""
    N, B = int(off[-1]), len(off) - 1
    owner = np.repeat(np.arange(B), np.diff(off))          # user of every flat row
    tiles = []
    for g in range((N + seg - 1) // seg):
        lo, hi = g * seg, min((g + 1) * seg, N)
        r = lo
        while r < hi:
            u = owner[r]
            piece_end = min(int(off[u + 1]), hi)
            t = r
            while t < piece_end:
                n = min(32, piece_end - t)
                tiles.append((g, u, t, n))
                t += n
            r = piece_end
    return np.array(tiles, dtype=np.int64).reshape(-1, 4)


@pytest.mark.parametrize("lens,seg", [
    ([700, 0, 1, 31, 32, 33, 2100, 64, 0, 95, 1029], 64),
    ([700, 0, 1, 31, 32, 33, 2100, 64, 0, 95, 1029], 992),
    ([700, 0, 1, 31, 32, 33, 2100, 64, 0, 95, 1029], 0),
    ([0, 0, 5], 32),
    ([1], 0),
    ([0, 0, 0], 0),
    ([40000, 3, 0, 0, 977, 12345], 4096),
])
def test_schedule_is_the_brute_force_tiling(lens, seg):
    off = I.offsets_from_lengths(lens)
    d_ = desc(len(lens), int(off[-1]), seg)
    got = V.vista_summarize_schedule(d_, off)
    want = brute_force_tiles(off, V.vista_summarize_segment_items(d_))
    assert np.array_equal(got, want)
    covered = np.zeros(int(off[-1]), dtype=np.int32)        # every row exactly once, under its own user
    for g, u, r, n in got:
        covered[r:r + n] += 1
        assert off[u] <= r and r + n <= off[u + 1]
    assert np.all(covered == 1)


def test_schedule_of_the_jagged_workload():
    c = I.CONFIGS[2]
    off = I.offsets_from_lengths(I.lengths(c))
    d_ = desc(c.B, int(off[-1]))
    got = V.vista_summarize_schedule(d_, off)
    assert np.array_equal(got, brute_force_tiles(off, V.vista_summarize_segment_items(d_)))
    assert got[:, 3].sum() == off[-1]


@pytest.mark.parametrize("seed", range(6))
def test_schedule_stays_in_bounds_for_any_offsets(seed):
    """Offsets that are decreasing, all zero, negative or beyond N: what the kernels walk is
    wrong but every tile stays inside [0, N) and every user index inside [0, B)."""
    g = np.random.default_rng(seed)
    B, N = 9, 5000
    kinds = [
        g.integers(-3 * N, 3 * N, size=B + 1),
        np.zeros(B + 1, dtype=np.int64),
        np.full(B + 1, 10 * N),
        np.sort(g.integers(0, N, size=B + 1))[::-1].copy(),
        np.concatenate([[0], np.sort(g.integers(0, 2 * N, size=B))]),
        np.concatenate([[7], g.integers(0, N, size=B - 1), [N]]),
    ]
    for off in kinds:
        for seg in (32, 256, 4096):
            t = V.vista_summarize_schedule(desc(B, N, seg), off.astype(np.int64))
            if len(t) == 0:
                continue
            assert t[:, 1].min() >= 0 and t[:, 1].max() < B
            assert t[:, 2].min() >= 0 and (t[:, 2] + t[:, 3]).max() <= N
            assert t[:, 3].min() >= 1 and t[:, 3].max() <= 32
            assert np.all(t[:, 2] >= t[:, 0] * seg) and np.all(t[:, 2] + t[:, 3] <= (t[:, 0] + 1) * seg)
            assert len(t) <= N + B * ((N + seg - 1) // seg)      # the walk ends


def test_schedule_rejects_bad_arguments():
    import ctypes as C
    L = V.lib()
    d_ = desc(2, 100)
    assert L.vista_summarize_schedule(C.byref(d_), None, None, 0) == -1
    off = np.array([0, 50, 100], dtype=np.int64)
    ptr = off.ctypes.data_as(C.POINTER(C.c_int64))
    assert L.vista_summarize_schedule(C.byref(d_), ptr, None, 5) == -1
    assert L.vista_summarize_schedule(C.byref(desc(0, 100)), ptr, None, 0) == -1
    assert L.vista_summarize_schedule(C.byref(d_), ptr, None, 0) == 4        # 50 rows = 2 tiles per user


@pytest.mark.parametrize("kw,base,call", [
    (dict(B=64, N=768597), 3008, 3008),
    (dict(B=8, N=8_000_000), 7840, 31264),                       # 256 segments instead of 1024
    (dict(B=1, N=7001), 256, 128),
    (dict(B=256, N=14_026_438, S=512, d=256, H=8), 7840, 31328), # 448 segments of four head groups: seven turns of 256
    (dict(B=8, N=8_000_000, seg=4096), 4096, 4096)])
def test_the_segment_size_a_call_uses(kw, base, call):
    d_ = desc(**kw)
    assert V.vista_summarize_segment_items(d_) == base
    assert V.vista_summarize_call_segment_items(d_) == call
    stated = V.vista_summarize_workspace_bytes(d_)
    assert V.vista_summarize_call_segment_items(d_, stated) == call
    least = V.vista_summarize_workspace_bytes(desc(**{**kw, "seg": base}))
    assert V.vista_summarize_call_segment_items(d_, least) == (base if least < stated else call)
    assert V.vista_summarize_call_segment_items(d_, least - 1) == 0
    off = np.linspace(0, kw["N"], kw["B"] + 1).astype(np.int64)
    given = desc(**{**kw, "seg": call})
    assert np.array_equal(V.vista_summarize_schedule(given, off), brute_force_tiles(off, call))


def test_the_segment_size_of_an_invalid_call():
    assert V.vista_summarize_call_segment_items(desc(0, 100)) == 0
    assert V.vista_summarize_call_segment_items(desc(2, 100), 1) == 0


@pytest.mark.parametrize("form", ["softmax", "silu"])
@pytest.mark.parametrize("d,H", [(128, 4), (256, 8)])
@pytest.mark.parametrize("S", [64, 128, 256, 512])
@pytest.mark.parametrize("own", [False, True])
def test_where_a_history_is_short(form, d, H, S, own):
    """Workgroups of half the heads are twice as many, so the segments that fill the chip with them are twice as long: the
    segment size tells which kind a call takes.  Many users make a history long."""
    told = 0
    for B in (1, 2, 3, 5, 8, 13, 30, 60, 100, 200):
        edge = short_history_limit(form, d, S) - user_as_items(form, d, S, own) * (B - 1)
        for N in (edge - 999, edge, edge + 1, edge + 999):
            if N <= always_short(d, S):
                continue
            assert is_short_history(form, d, S, N, B, own) == (N <= edge)
            q = V.summarize_desc(B, S, d, H, V.VISTA_BF16, N, own, attn=V.VISTA_ATTN_SILU if form == "silu" else V.VISTA_ATTN_SOFTMAX)
            seg = fitted_segment(form, d, S, N, B, own)
            base = V.vista_summarize_segment_items(q)                                 # what stays where the records are too many
            fits = (-(-N // seg) + B) * H * (S // 32) * 18 * 256 < 63 << 20 or seg >= base
            assert V.vista_summarize_call_segment_items(q) == (seg if fits else base), (B, N)
            told += fits and seg != fitted_segment(form, d, S, N, 10 ** 6 if N <= edge else 0, own)
    assert told >= 4


@pytest.mark.parametrize("form", ["softmax", "silu"])
@pytest.mark.parametrize("S", [64, 128, 256])
@pytest.mark.parametrize("own", [False, True])
def test_where_a_workgroup_takes_one_head(form, S, own):
    """At d = 128 the heads of a segment are four workgroups instead of two or one, so the segments that fill the chip are longer: the
    size tells on which side of the limit a call is.  (At d = 256 and at 512 seeds halves are as many.)"""
    told = 0
    for B in (1, 2, 5, 17, 64, 200):
        lo, hi = 1024, 10 ** 6                                        # takes_one_head falls once
        assert takes_one_head(form, 128, S, lo, B, own) and not takes_one_head(form, 128, S, hi, B, own)
        while hi - lo > 1:
            mid = (lo + hi) // 2
            lo, hi = (mid, hi) if takes_one_head(form, 128, S, mid, B, own) else (lo, mid)
        for N in (lo - 999, lo, hi, hi + 999):
            q = V.summarize_desc(B, S, 128, 4, V.VISTA_BF16, N, own, attn=V.VISTA_ATTN_SILU if form == "silu" else V.VISTA_ATTN_SOFTMAX)
            assert V.vista_summarize_call_segment_items(q) == fitted_segment(form, 128, S, N, B, own), (B, N)
        told += fitted_segment(form, 128, S, lo, B, own) != fitted_segment(form, 128, S, hi, B, own)
    assert told >= 3
