"""The one-wave forward where its shortcuts could show: values that are not
finite, entries outside [0, N), heads that fall to either kernel in one call
(uneven lists, large-magnitude blocks), and rows of a few entries among paced
ones.

The same heads computed in one call (one-wave: 2,048 rows and up) and in two
halves (two-wave); test_gpu_wave.py derives the tolerance."""
import numpy as np
import pytest
import torch

from parity import MAX_ABS, REL_L2, ULP_REL, value_errors
from test_gpu_wave import forward, one_wave_heads, slice_lists
from workload import Problem

pytestmark = pytest.mark.gpu

INF, NAN = float("inf"), float("nan")


def halves(p, q, k, v, rp, ci, training):
    h, hkv, out = p.heads_q // 2, p.heads_kv // 2, []
    ph = p.replace(heads_q=h, heads_kv=hkv)
    for i in range(2):
        r, c = slice_lists(dict(row_ptr=rp, col_idx=ci), p.N_joint, i * h, (i + 1) * h)
        cut = [t[:, i * s:(i + 1) * s].contiguous() for t, s in ((q, h), (k, hkv), (v, hkv))]
        o, lse, even = forward(ph, *cut, r, c, training)
        assert even is None
        out.append((o, lse))
    return [np.concatenate([a[j] for a in out], 1) for j in range(2)]


def assert_same(got, want):
    """Equal where not finite (any NaN for NaN), within the bar elsewhere."""
    (o, lse), (o2, lse2) = got, want
    assert np.array_equal(np.isnan(o), np.isnan(o2)), "NaN at %d and %d values" % (np.isnan(o).sum(), np.isnan(o2).sum())
    inf = np.isinf(o2)
    assert np.array_equal(np.isinf(o), inf) and np.array_equal(o[inf], o2[inf])
    fin = np.isfinite(o2)
    _, beyond, rel = value_errors(o[fin], o2[fin], 2 * ULP_REL["bf16"])
    assert beyond <= 2 * MAX_ABS and rel <= REL_L2, (beyond, rel)
    assert np.array_equal(np.isnan(lse), np.isnan(lse2)) and np.array_equal(np.isinf(lse), np.isinf(lse2))
    fin = np.isfinite(lse2)
    assert np.array_equal(np.sign(lse[np.isinf(lse)]), np.sign(lse2[np.isinf(lse)]))
    assert np.abs(lse[fin] - lse2[fin]).max() <= 2e-5 * max(1.0, np.abs(lse2[fin]).max())


def lists_of(rows, device="cuda"):
    """CSR of a list of int arrays."""
    rp = np.concatenate([[0], np.cumsum([len(r) for r in rows])]).astype(np.int32)
    return torch.from_numpy(rp).to(device), torch.from_numpy(np.concatenate(rows).astype(np.int32)).to(device)


def inputs(p, seed):
    """Q, K, V in bf16, N(0, 1) (padding tokens too: they may hold anything finite)."""
    g = torch.Generator(device="cuda").manual_seed(seed)
    return [torch.randn((p.batch, h, p.L_joint, p.head_dim), generator=g, device="cuda").bfloat16()
            for h in (p.heads_q, p.heads_kv, p.heads_kv)]


def random_rows(p, k, seed):
    g = np.random.default_rng(seed)
    return [np.sort(g.choice(p.N, k, replace=False)) for _ in range(p.heads_q * p.N)]


# problems that the one-wave kernel takes: 352 blocks unpadded, 352 and (for training) 900 with cut cubes
FLAT = Problem(1, 6, 6, 128, 16, 44, 32, dtype=1)
CUT = {False: Problem(1, 6, 6, 128, 15, 42, 30, dtype=1), True: Problem(1, 4, 4, 128, 18, 58, 46, dtype=1)}
LEN = 50                       # entries a row, long enough for either


def poison(what, q, k, v):
    """Puts values that are not finite into the second head of each half."""
    blk = lambda n: slice(64 * n, 64 * n + 64)
    for h in (1, q.shape[1] // 2 + 1):
        if what == "nan-query":
            q[0, h, 69, 17] = NAN                      # one query of block 1
        elif what == "inf-query":
            q[0, h, 69, 17] = INF
        elif what == "nan-key-block":
            k[0, h, blk(0)] = NAN                      # first in every list that holds it
        elif what == "nan-key":
            k[0, h, 64 * 5 + 40, 3] = NAN
        elif what == "inf-keys":
            k[0, h, 0:32, 3] = INF                     # half a block: scores of +inf and -inf
        elif what == "inf-keys-late":
            k[0, h, 64 * 20:64 * 20 + 32, 3] = -INF
        elif what == "all-scores-infinite":
            k[0, h, :, 3] = INF
        elif what == "nan-value":
            v[0, h, 64 * 6 + 1, 9] = NAN
        elif what == "inf-value":
            v[0, h, 64 * 6 + 1, 9] = -INF


@pytest.mark.parametrize("training", [False, True])
@pytest.mark.parametrize("what", ["nan-query", "inf-query", "nan-key-block", "nan-key", "inf-keys", "inf-keys-late",
                                  "all-scores-infinite", "nan-value", "inf-value"])
def test_values_that_are_not_finite_pass_as_in_the_two_wave_kernel(what, training):
    """A NaN is never turned into a number, an infinite score has weight 0 or
    makes its row NaN, and other rows are untouched."""
    for p in (FLAT, CUT[training]):
        q, k, v = inputs(p, 91)
        rp, ci = lists_of(random_rows(p, LEN, 92))
        poison(what, q, k, v)
        print("\n[%s] %s" % (what, p), flush=True)
        o, lse, even = forward(p, q, k, v, rp, ci, training)
        assert np.array_equal(even, one_wave_heads(p, rp, (q, k, v) if training else None))
        # in training, a head whose key blocks are all flagged is the two-wave kernel's
        assert (even == LEN).sum() == p.heads_q - (2 if training and what == "all-scores-infinite" else 0)
        want = halves(p, q, k, v, rp, ci, training)
        assert (~np.isfinite(want[0])).any()
        assert_same((o, lse), want)


@pytest.mark.parametrize("training", [False, True])
def test_entries_outside_the_range_read_nothing(training):
    """Entries outside [0, N) at the first, middle and last places, in a head
    whose block 0 (in no list) holds infinities and NaN: finite, and as the
    lists without those entries give."""
    for p in (FLAT, CUT[training]):
        q, k, v = inputs(p, 93)
        blk0 = slice(0, 64)
        k[:, :, blk0] = NAN
        v[:, ::2, blk0] = INF
        v[:, 1::2, blk0] = NAN
        g = np.random.default_rng(94)
        rows, holes = [], []
        for i in range(p.heads_q * p.N):
            r = np.sort(1 + g.choice(p.N - 1, LEN, replace=False))
            rows.append(r)
            bad = [-1, p.N, 2 ** 30, -2 ** 31]
            h = np.insert(r, [0, 8], [bad[i % 4], bad[(i + 1) % 4]])
            holes.append(np.append(h, bad[(i + 2) % 4]) if i % 2 else h)
        rows[5], holes[5] = rows[5][:0], np.full(LEN + 2, -1)          # a row of nothing else
        rp, ci = lists_of(holes)
        o, lse, even = forward(p, q, k, v, rp, ci, training)
        assert (even > 0).all()
        assert np.isfinite(o).all() and not np.isnan(lse).any()
        # the same lists without the entries, on a head count below the rule: two-wave
        want = halves(p, q, k, v, *lists_of(rows), training)
        assert_same((o, lse), want)
        row5 = slice(5 * 64, 6 * 64)
        assert (o[0, 0, row5] == 0).all() and np.isneginf(lse[0, 0, row5]).all()


@pytest.mark.parametrize("training", [False, True])
def test_heads_of_both_kernels_in_one_call(training):
    """Every other head has uneven lists (12 to 88 entries) and stays with the
    two-wave kernel; one head is even but for an eighth of its rows, one has one
    more such row."""
    for p in (FLAT, CUT[training]):
        q, k, v = inputs(p, 95)
        g = np.random.default_rng(96)
        rows = random_rows(p, LEN, 97)
        for h in range(1, p.heads_q, 2):
            for i in range(h * p.N, (h + 1) * p.N):
                rows[i] = np.sort(g.choice(p.N, int(g.integers(12, 89)), replace=False))
        # heads at the edge of the rule: long rows (the average, LEN + 1/2, is what
        # counts; LEN + 4 is more than 1/16 off it)
        for h, n in ((0, p.N // 8), (2, p.N // 8 + 1)):
            for i in range(h * p.N, h * p.N + n):
                rows[i] = np.sort(g.choice(p.N, LEN + 4, replace=False))
        rp, ci = lists_of(rows)
        o, lse, even = forward(p, q, k, v, rp, ci, training)
        want_even = one_wave_heads(p, rp)
        assert np.array_equal(even > 0, want_even > 0) and np.allclose(even, want_even, rtol=1e-6)
        assert even[0] > 0 and even[2] == 0 and not (even[1::2] > 0).any() and (even[4::2] > 0).all()
        assert_same((o, lse), halves(p, q, k, v, rp, ci, training))


def test_heads_with_large_magnitude_blocks():
    """Training: two-term P in the one-wave kernel where few blocks are flagged;
    from 0.7 flagged key blocks an average list, or from half of the query
    blocks, the head is the two-wave kernel's."""
    for p in (FLAT, CUT[True]):
        q, k, v = inputs(p, 101)
        rp, ci = lists_of(random_rows(p, LEN, 102))
        g = np.random.default_rng(103)
        most = int(0.7 * p.N / LEN)
        flag = lambda x, h, n: [x[0, h, 64 * i + 21].mul_(12) for i in g.choice(p.N, n, replace=False)]
        flag(k, 0, most)
        flag(v, 1, most + 1)
        flag(q, 2, p.N // 2)
        flag(q, 3, p.N // 2 + 1)
        o, lse, even = forward(p, q, k, v, rp, ci, True)
        want = one_wave_heads(p, rp, (q, k, v))
        assert np.array_equal(even, want) and [x > 0 for x in even[:4]] == [True, False, True, False]
        assert_same((o, lse), halves(p, q, k, v, rp, ci, True))
        _, _, plain = forward(p, q, k, v, rp, ci, False)               # inference: one-term P everywhere
        assert (plain == LEN).all()


@pytest.mark.parametrize("training", [False, True])
def test_rows_of_few_entries_among_paced_ones(training):
    """Rows of 0, 1, 2, 3, 63, 64 and 65 entries and of every block, spread over
    even heads: the pipeline without its loop, a list window's edges, and walks
    that are not paced."""
    for p in (FLAT, CUT[training]):
        q, k, v = inputs(p, 98)
        g = np.random.default_rng(99)
        rows = random_rows(p, LEN, 100)
        odd = [0, 1, 2, 3, 63, 64, 65, p.N]
        for h in range(p.heads_q):
            for j, n in enumerate(g.choice(p.N, 24, replace=False)):
                rows[h * p.N + n] = np.sort(g.choice(p.N, odd[(h + j) % len(odd)], replace=False))
        rp, ci = lists_of(rows)
        o, lse, even = forward(p, q, k, v, rp, ci, training)
        assert (even > 0).all() and np.allclose(even, one_wave_heads(p, rp), rtol=1e-6)
        assert_same((o, lse), halves(p, q, k, v, rp, ci, training))
