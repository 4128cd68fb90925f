"""The encoder of the bulk build at the values where its search can go wrong: ties at either end (the lowest
channel is the outlier), an end on every channel, zeros of both signs, equal values, infinities, NaN."""
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
