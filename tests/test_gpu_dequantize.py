"""qaq_dequantize at the edges of its work items (runs of eight channels, units of 16 tokens, half-units of
8, tiles of 256 positions) for every width class, outlier count and a range that starts and ends inside a
tile: bit-exact against the oracle's reconstruction rounded to fp16."""
import numpy as np
import pytest

from paper_2403_04643_amd import qaq, workloads as W
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


@pytest.mark.parametrize("head_dim,context,n_o,widths", [(64, 300, 1, (2, 3, 4, 8)), (128, 257, 3, (1, 2, 3, 4, 8)), (128, 40, 0, (4, 8))])
@pytest.mark.parametrize("shift", [1, 2, 4, 7])
def test_outputs_at_any_fp16(head_dim, context, n_o, widths, shift):
    """Outputs that start `shift` halves into a buffer, as slices of a caller's larger tensors do: the same numbers as
    at the buffer's start, and nothing beside them."""
    import torch
    sh = W.shape(1, batch=1, n_q_heads=2, n_kv_heads=2, head_dim=head_dim, context=context)
    print(f"dequantize {sh} n_o={n_o} widths={widths} shift={shift}", flush=True)
    K, V = W.make_kv(1, sh)
    rng = np.random.default_rng(context + shift)
    bk, bv = (rng.choice(np.array(widths, np.uint8), size=K.shape[:3]) for _ in range(2))
    oc, gc = make_pair(sh, 0.02, n_outlier_per_side=n_o, bit_set=(1, 2, 3, 4, 8))
    oc.append(K, V, bk, bv)
    gc.quantize_append(dev(K), dev(V), dev(bk), dev(bv))
    t0, t1 = context // 5, context - 1
    n = 2 * (t1 - t0) * head_dim
    outs = [torch.full((n + 16,), -7.0, dtype=torch.float16, device="cuda") for _ in range(2)]
    stream = torch.cuda.current_stream().cuda_stream
    assert gc.lib.qaq_dequantize(gc.h, t0, t1, outs[0].data_ptr() + 2 * shift, outs[1].data_ptr() + 2 * shift, stream) == qaq.OK
    for out, ref in zip(outs, oc.dequantize()):
        got = out.cpu().numpy()
        want = np.ascontiguousarray(ref.astype(F16)[:, :, t0:t1])
        np.testing.assert_array_equal(got[shift:shift + n].view(np.uint16), want.reshape(-1).view(np.uint16))
        assert (got[:shift] == -7.0).all() and (got[shift + n:] == -7.0).all()
