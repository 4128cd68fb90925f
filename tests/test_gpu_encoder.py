"""The encoder of the bulk build at the values where its search can go wrong: ties at either end (the lowest
channel is the outlier), an end on every channel, zeros of both signs, equal values, infinities, NaN, thresholds that
are no fp16 number.

A wavefront encodes sixteen tokens of an append together and has two searches: a short one where all of them allow it
and a general one else.  Kinds of tokens are therefore laid out by whole groups of sixteen where the short search is
meant, and the tests count the groups."""
import numpy as np
import pytest

from paper_2403_04643_amd import workloads as W
from tests.parity_util import F16, compare_canonical, dev, make_pair

pytestmark = pytest.mark.gpu


def _edge_tokens(rng, n, D):
    """[n, D] fp16, kind by position."""
    x = (rng.standard_normal((n, D)) * 2).astype(F16)
    for t in range(n):
        kind = t % 8
        if kind == 0:                                   # both ends on channels that walk over the vector
            x[t] = rng.integers(-3, 4, size=D)
            x[t, (t // 8) % D] = 9.0
            x[t, (t // 8 * 5 + 3) % D] = -9.0 if (t // 8 * 5 + 3) % D != (t // 8) % D else 9.0
        elif kind == 1:                                 # ties everywhere
            x[t] = rng.integers(-1, 2, size=D)
        elif kind == 2:                                 # the largest value a zero of either sign
            x[t] = -np.abs(x[t])
            x[t, rng.integers(0, D, size=3)] = 0.0
            x[t, rng.integers(0, D, size=3)] = -0.0
        elif kind == 3:                                 # the smallest
            x[t] = np.abs(x[t])
            x[t, rng.integers(0, D, size=3)] = -0.0
        elif kind == 4:
            x[t] = [0.0, -0.0, 1.5, -65504.0][t // 8 % 4]
        elif kind == 5:                                 # one value differs
            x[t] = 0.25
            x[t, t // 8 % D] = 0.25 + (1 if t % 16 < 8 else -1) * 0.125
        elif kind == 6:                                 # subnormal numbers
            x[t] = rng.integers(-40, 41, size=D) * F16(6e-8)
    return x


@pytest.mark.parametrize("head_dim,bit_set,n_o", [(128, (2, 3, 4, 8), 1), (64, (2, 3, 4, 8), 1), (128, (1, 2, 3, 4, 8), 1),
                                                  (128, (2, 4), 1), (128, (2, 3, 4, 8), 3), (64, (2, 3, 4, 8), 2), (128, (2, 3, 4, 8), 0)])
def test_ends_of_a_token(head_dim, bit_set, n_o):
    n = 8 * 2 * head_dim + 70                           # whole tiles and a part, every channel an end
    sh = W.shape(2, batch=1, n_q_heads=1, n_kv_heads=1, head_dim=head_dim, context=n)
    print(f"encoder: D={head_dim} set={bit_set} n_o={n_o}", flush=True)
    rng = np.random.default_rng(23)
    K, V = (_edge_tokens(rng, n, head_dim)[None, None] for _ in range(2))
    cut = 300
    for given in (False, True):
        bits = [rng.choice(np.array(bit_set, np.uint8), size=(1, 1, n)) if given else None for _ in range(2)]
        oc, gc = make_pair(sh, 0.02, bit_set=bit_set, n_outlier_per_side=n_o)
        for lo, hi in ((0, cut), (cut, n)):
            part = [None if b is None else b[:, :, lo:hi] for b in bits]
            oc.append(K[:, :, lo:hi], V[:, :, lo:hi], *part)
            gc.quantize_append(dev(K[:, :, lo:hi]), dev(V[:, :, lo:hi]), *[None if b is None else dev(b) for b in part])
        compare_canonical(oc, gc, f"given={given}")


@pytest.mark.parametrize("head_dim", [128, 64])
def test_values_that_are_not_numbers(head_dim):
    """An infinity or a NaN at an end is an outlier; the rest of the token is as if a large number stood there.  A NaN's
    code is the top one, like an infinity's."""
    n = 90
    sh = W.shape(2, batch=1, n_q_heads=1, n_kv_heads=1, head_dim=head_dim, context=n)
    rng = np.random.default_rng(29)
    base = (rng.standard_normal((1, 1, n, head_dim)) * 2).astype(F16)
    ch = rng.integers(0, head_dim, size=n)
    out = []
    for put in (F16(60000.0), F16(np.inf), F16(np.nan)):
        x = base.copy()
        x[0, 0, np.arange(n), ch] = put
        _, gc = make_pair(sh, 0.02)
        gc.quantize_append(dev(x), dev(x))
        out.append({k: v.cpu().numpy() for k, v in gc.export_canonical(0).items()})
        val = out[-1]["oval"][0, 0][out[-1]["oidx"][0, 0] == ch[:, None]]
        np.testing.assert_array_equal(val.view(np.uint16), np.full(n, put).view(np.uint16))
    for key in ("bits", "oidx", "codes", "minmax"):
        a, b, c = (o[key].view(np.uint16) if key == "minmax" else o[key] for o in out)
        np.testing.assert_array_equal(a, b, err_msg=key)
        np.testing.assert_array_equal(a, c, err_msg=key)


# ---- whole wavefronts on the short search, and whole wavefronts sent to the general one by a single token ----

GROUP = 16          # tokens of a wavefront


def _groups_with(flag):
    """flag [n] per token -> per whole group of sixteen: all of them."""
    n = len(flag) // GROUP * GROUP
    return flag[:n].reshape(-1, GROUP).all(1)


def _ordinary_tokens(rng, n, D):
    """[n, D] fp16 whose largest and smallest values are finite and not zero, kind by position."""
    x = np.zeros((n, D), F16)
    for t in range(n):
        kind, i = t % 8, t // 8
        a, b = i % D, (i * 5 + 3) % D
        b = b if b != a else (b + 1) % D
        if kind == 0:                                   # both ends on channels that walk over the vector
            x[t] = rng.integers(-3, 4, size=D)
            x[t, a], x[t, b] = 9.0, -9.0
        elif kind == 1:                                 # many channels tie at both ends, the lowest of them walking
            x[t] = rng.integers(-1, 2, size=D)
            x[t, : min(a, D - 2)] = 0.0
            x[t, -1 - i % 2], x[t, -2 + i % 2] = 1.0, -1.0
        elif kind == 2:                                 # all values equal
            x[t] = [1.5, -65504.0, 6e-8, -0.25][i % 4]
        elif kind == 3:                                 # one value differs
            x[t] = 0.25
            x[t, a] = 0.375 if i % 2 else 0.125
        elif kind == 4:                                 # subnormal numbers
            x[t] = rng.integers(-40, 41, size=D) * F16(6e-8)
            x[t, a], x[t, b] = 41 * F16(6e-8), -41 * F16(6e-8)
        elif kind == 5:                                 # zeros of both signs between the ends: an empty range
            x[t] = np.where(rng.random(D) < 0.5, F16(0.0), F16(-0.0))
            x[t, a], x[t, b] = 2.0, -2.0
        elif kind == 6:                                 # ends far outside a range of one or two subnormal steps
            x[t] = rng.integers(0, 2 + i % 2, size=D) * F16(6e-8)
            x[t, a], x[t, b] = 65504.0, -65504.0
        else:
            x[t] = rng.standard_normal(D) * 2
            x[t, a], x[t, b] = 12.0, -12.0
    return x


def _append_in_two(oc, gc, K, V, cut, bits):
    n = K.shape[2]
    for lo, hi in ((0, cut), (cut, n)):
        part = [None if b is None else b[:, :, lo:hi] for b in bits]
        oc.append(K[:, :, lo:hi], V[:, :, lo:hi], *part)
        gc.quantize_append(dev(K[:, :, lo:hi]), dev(V[:, :, lo:hi]), *[None if b is None else dev(b) for b in part])


@pytest.mark.parametrize("head_dim,bit_set", [(128, (2, 3, 4, 8)), (64, (2, 3, 4, 8)), (128, (1, 2, 3, 4, 8)), (64, (2, 4))])
def test_ends_on_the_short_search(head_dim, bit_set):
    n = 8 * 2 * head_dim + 70
    sh = W.shape(2, batch=1, n_q_heads=1, n_kv_heads=1, head_dim=head_dim, context=n)
    print(f"encoder, short search: D={head_dim} set={bit_set}", flush=True)
    rng = np.random.default_rng(31)
    K, V = (_ordinary_tokens(rng, n, head_dim)[None, None] for _ in range(2))
    for x in (K, V):
        x[0, 0, 3 * GROUP + 5 :: 8 * GROUP] = 0.0            # one group in eight has a token that the short search cannot take
    for x in (K, V):
        ends = np.stack([x[0, 0].max(1), x[0, 0].min(1)]).astype(np.float32)
        short = _groups_with((np.isfinite(ends) & (ends != 0)).all(0))
        assert 0.8 < short.mean() < 0.95
    for given in (False, True):
        bits = [rng.choice(np.array(bit_set, np.uint8), size=(1, 1, n)) if given else None for _ in range(2)]
        oc, gc = make_pair(sh, 0.02, bit_set=bit_set)
        _append_in_two(oc, gc, K, V, 256 + 3 * GROUP, bits)   # (the second append's groups start on its first token)
        compare_canonical(oc, gc, f"given={given}")


_ALL = np.sort(np.concatenate([np.arange(0x0000, 0x7c01), np.arange(0x8001, 0xfc01)]).astype(np.uint16).view(F16).astype(np.float32))
_UP, _DOWN = np.float32(np.inf), np.float32(-np.inf)
THRESHOLDS = [                                            # (lo, hi)
    (-1.5, 1.5),                                          # fp16 numbers: a value on one is no outlier
    (np.nextafter(np.float32(-1.5), _UP), np.nextafter(np.float32(1.5), _DOWN)),      # inside of them
    (np.nextafter(np.float32(-1.5), _DOWN), np.nextafter(np.float32(1.5), _UP)),      # outside
    (-65504.0, 65504.0), (-70000.0, 70000.0), (-1e30, 1e30),                           # only an infinity is outside
    (-65500.0, 65500.0),                                  # rounds to the largest fp16 number
    (-1e-9, 1e-9), (1e-9, 1.0), (-1.0, -1e-9),            # between zero and the smallest number; a zero is outside of the last two
    (0.0, 2.0), (-2.0, -0.0),                             # the border a zero, values of the other sign outside
    (-9e-8, 9e-8),                                        # between subnormal numbers
]


def _threshold_tokens(rng, n, D, lo, hi, cap):
    """[n, D] fp16 and the number of values above and below per token: as many as are kept at most, but in every
    fourth group of sixteen, where up to four more are."""
    lo, hi = np.float32(lo), np.float32(hi)
    below, inside, above = _ALL[_ALL < lo], _ALL[(_ALL >= lo) & (_ALL <= hi)], _ALL[_ALL > hi]
    x = np.zeros((n, D), F16)
    counts = np.zeros((n, 2), int)
    for t in range(n):
        near = np.concatenate([inside[:3], inside[-3:]])
        body = np.where(rng.random(D) < 0.2, rng.choice(near, size=D), rng.choice(inside, size=D))
        if t % 3 == 0:
            body = np.where(body == 0, F16(-0.0), body)
        most = cap + (4 if t // GROUP % 4 == 3 else 0)
        k = [int(rng.integers(0, most + 1)), int(rng.integers(0, most + 1))] if t % 5 else [most, most]
        spread = body.max() > body.min()
        if np.isinf(above).all():                                 # (more infinities than are kept leave no range)
            k = [min(k[0], cap), min(k[1], cap)]
        ch = rng.permutation(D)[: k[0] + k[1]]
        for j in range(k[0] + k[1]):
            out = above if j < k[0] else below[::-1]              # nearest the threshold first
            first = j == 0 or j == k[0]
            if np.isinf(out[0]):
                body[ch[j]] = out[0]
            elif first and t % 7 == 0 and spread:
                body[ch[j]] = out[-1]                             # the infinity (a code of it is defined where there is a range)
            else:
                body[ch[j]] = out[rng.integers(0, 2 if t % 2 else len(out) - 1) if len(out) > 2 else 0]
        x[t] = body
        counts[t] = k
    return x, counts


@pytest.mark.parametrize("head_dim,cap,bit_set", [(128, 4, (2, 3, 4, 8)), (64, 2, (2, 3, 4, 8)), (128, 1, (1, 2, 3, 4, 8)), (64, 3, (2, 4))])
def test_thresholds_at_their_edges(head_dim, cap, bit_set):
    n, H = 500, len(THRESHOLDS)
    sh = W.shape(2, batch=1, n_q_heads=H, n_kv_heads=H, head_dim=head_dim, context=n)
    print(f"encoder, thresholds: D={head_dim} cap={cap} set={bit_set}", flush=True)
    rng = np.random.default_rng(37)
    K, V = np.zeros((1, H, n, head_dim), F16), np.zeros((1, H, n, head_dim), F16)
    full = []
    for h, (lo, hi) in enumerate(THRESHOLDS):
        for x in (K, V):
            x[0, h], counts = _threshold_tokens(rng, n, head_dim, lo, hi, cap)
            xf = x[0, h].astype(np.float32)
            np.testing.assert_array_equal(np.stack([(xf > np.float32(hi)).sum(1), (xf < np.float32(lo)).sum(1)], 1), counts)
            full.append(_groups_with((counts <= cap).all(1)))
    assert 0.7 < np.mean(full) < 0.95                          # groups that one sweep serves; the others go value by value
    thr = np.array([THRESHOLDS, THRESHOLDS], np.float32)
    for given in (False, True):
        bits = [rng.choice(np.array(bit_set, np.uint8), size=(1, H, n)) if given else None for _ in range(2)]
        oc, gc = make_pair(sh, 0.02, bit_set=bit_set, n_outlier_per_side=cap, outlier_thresholds=thr)
        _append_in_two(oc, gc, K, V, 256 + 3 * GROUP, bits)
        compare_canonical(oc, gc, f"given={given}")


@pytest.mark.parametrize("head_dim,n_o,thr", [(128, 1, None), (64, 1, None), (128, 3, None), (128, 4, (-2.5, 2.5)), (64, 2, (-2.5, 2.5))])
def test_a_value_that_is_not_a_number_concerns_its_token_only(head_dim, n_o, thr):
    """A NaN sends its wavefront to the general search, which must leave the other fifteen tokens what they are."""
    n = 300
    sh = W.shape(2, batch=1, n_q_heads=1, n_kv_heads=1, head_dim=head_dim, context=n)
    rng = np.random.default_rng(41)
    base = np.clip(rng.standard_normal((1, 1, n, head_dim)), -2.4, 2.4).astype(F16)
    for t in range(n):
        ch = rng.permutation(head_dim)[: n_o + 1]
        base[0, 0, t, ch[: t % (n_o + 1)]] = 3.0 + t % 5
        base[0, 0, t, ch[n_o]] = -4.0
    hit = np.arange(5, n, 2 * GROUP)
    x = base.copy()
    x[0, 0, hit, rng.integers(0, head_dim, size=len(hit))] = np.where(np.arange(len(hit)) % 2, np.nan, -np.nan).astype(F16)
    out = []
    for data in (base, x):
        _, gc = make_pair(sh, 0.02, n_outlier_per_side=n_o, outlier_thresholds=None if thr is None else [[thr], [thr]])
        gc.quantize_append(dev(data), dev(data))
        out.append([{k: v.cpu().numpy() for k, v in gc.export_canonical(side).items()} for side in (0, 1)])
    rest = np.setdiff1d(np.arange(n), hit)
    for side in (0, 1):
        for key in ("bits", "minmax", "oidx", "oval", "codes"):
            a, b = (np.ascontiguousarray(o[side][key][0, 0, rest]).view(np.uint8) for o in out)
            np.testing.assert_array_equal(a, b, err_msg=f"side {side} {key}")


@pytest.mark.parametrize("head_dim,n_o", [(128, 1), (64, 1), (128, 2)])
def test_sides_of_which_every_token_widens(head_dim, n_o):
    """Nothing of such a tile side's old codes is kept; of its neighbours, one token's are, or those of the tokens that
    were at the widest width already."""
    sh = W.shape(2, batch=1, n_q_heads=2, n_kv_heads=2, head_dim=head_dim, context=3 * 256 + 90)
    rng = np.random.default_rng(43)
    K, V = W.make_kv(2, sh)
    narrow = rng.choice(np.array([2, 3, 4], np.uint8), size=K.shape[:3])
    narrow[:, :, 2 * 256 + 5 : 3 * 256 : 7] = 8            # the third tile: some need not widen
    wide = np.full_like(narrow, 8)
    wide[:, :, 256 + 100] = narrow[:, :, 256 + 100]        # the second tile: one stays
    oc, gc = make_pair(sh, 0.02, n_outlier_per_side=n_o)
    oc.append(K, V, narrow, narrow); gc.quantize_append(dev(K), dev(V), dev(narrow), dev(narrow))
    oc.requantize(wide, wide, K, V); gc.requantize(dev(wide), dev(wide), dev(K), dev(V))
    compare_canonical(oc, gc, "widened")
