"""Decode-step update: tiles that every row of the window covers take its rows without a look at their ends, the others with one.
Both against the separate calls, over the window lengths, ways of storing the rows, query heads per KV head and lengths around a
tile border at which the sides change over."""
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from paper_2403_04643_amd import qaq  # noqa: E402


@pytest.mark.parametrize("window", [1, 2, 3, 4, 5, 6, 7, 8])
@pytest.mark.parametrize("store", ["fp32", "fp16", "bf16"])
@pytest.mark.parametrize("G", [1, 3, 6])
def test_rows_of_covered_tiles(window, store, G):
    B, Hkv, D, T = 2, 3, 64, 508           # two tiles; the second is covered by no row, some, and all of them
    print(f"window {window} {store} G={G}", flush=True)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(100 * window + G)
    rnd = lambda *s: torch.randn(s, device="cuda", generator=gen)  # noqa: E731
    mk = lambda: qaq.Cache(qaq.make_config(B, Hkv * G, Hkv, D, T + 20, [0.05] * Hkv, window=window, sigma_s_max=2e-4, sigma_x_max=0.02,  # noqa: E731
                                           window_fp16=store == "fp16", window_bf16=store == "bf16"))
    k, v = rnd(B, Hkv, T + 20, D).half(), rnd(B, Hkv, T + 20, D).half()
    k0, v0 = k[:, :, :T].contiguous(), v[:, :, :T].contiguous()
    fused, separate = mk(), mk()
    for c in (fused, separate):
        c.quantize_append(k0, v0)
    for j in range(14):
        n = T + j + 1
        # sharp rows, so that widths follow single rows as they come and go
        scores = torch.softmax(4.0 * rnd(B, Hkv * G, n), dim=-1)
        kn, vn = k[:, :, n - 1].contiguous(), v[:, :, n - 1].contiguous()
        got = fused.decode_update(scores, kn, vn, k, v, want_bits=True)
        separate.quantize_append(kn[:, :, None], vn[:, :, None])
        want = separate.select_bits(scores)
        separate.requantize(*want, k, v)
        for a, b in zip(got, want):
            assert torch.equal(a, b), f"widths of step {j}"
    assert len(torch.unique(want[1])) > 1, "the rules gave every value one width"
    for side in (0, 1):
        a, b = fused.export_canonical(side), separate.export_canonical(side)
        for key in ("bits", "codes", "oidx"):
            assert torch.equal(a[key], b[key]), key
