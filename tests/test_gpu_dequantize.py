"""qaq_dequantize at the edges of its work items (runs of eight channels, units of 16 tokens, half-units of
8, tiles of 256 positions) for every width class, outlier count and a range that starts and ends inside a
tile: bit-exact against the oracle's reconstruction rounded to fp16."""
import numpy as np
import pytest

from paper_2403_04643_amd import workloads as W
from tests.parity_util import F16, dev, make_pair

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("head_dim", [64, 128])
@pytest.mark.parametrize("context", [1, 15, 17, 255, 300])
@pytest.mark.parametrize("n_o,widths", [(1, (2, 3, 4, 8)), (0, (2, 3, 4, 8)), (3, (1, 2, 3, 4, 8)), (1, (8,)), (4, (1, 4))])
def test_every_class_and_range(head_dim, context, n_o, widths):
    sh = W.shape(1, batch=2, n_q_heads=3, n_kv_heads=3, head_dim=head_dim, context=context)
    print(f"dequantize {sh} n_o={n_o} widths={widths}", flush=True)
    K, V = W.make_kv(1, sh)
    rng = np.random.default_rng(context + head_dim)
    bk, bv = (rng.choice(np.array(widths, np.uint8), size=K.shape[:3]) for _ in range(2))
    oc, gc = make_pair(sh, 0.02, n_outlier_per_side=n_o, bit_set=(1, 2, 3, 4, 8))
    oc.append(K, V, bk, bv)
    gc.quantize_append(dev(K), dev(V), dev(bk), dev(bv))
    want = [x.astype(F16).view(np.uint16) for x in oc.dequantize()]
    for t0, t1 in {(0, context), (context // 3, context), (context // 2, (context + context // 2 + 1) // 2)}:
        if t1 > t0:
            for got, ref in zip(gc.dequantize(t0, t1), want):
                np.testing.assert_array_equal(got.cpu().numpy().view(np.uint16), ref[:, :, t0:t1])
