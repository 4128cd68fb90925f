"""Attention where several workgroups read one KV head's codes: whichever order they are dealt to the dies in, every
(sequence, query head, part) is worked on once.  Shapes with parts in multiples of eight and not, with groups that fill
eight dies and with some left over, in both forms of the two-kernel scan."""
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from paper_2403_04643_amd import qaq  # noqa: E402
from tests.parity_util import attention_route  # noqa: E402

# K^ and V^ reach the reference rounded to fp16 (2^-11 of each value; logits of a few units, so at most about 1e-3 of a
# weight, and as much of the output); the library's own sums are off by 1e-5
TOL = 5e-3


@pytest.mark.parametrize("B,Hkv,G,D,T,kw,passes", [
    (8, 4, 6, 128, 1500, dict(n_outlier_per_side=2), False),                      # 5 parts of 6 tiles, groups of 48 workgroups without a rest
    (3, 7, 5, 64, 2600, dict(n_outlier_per_side=2), False),                       # 9 parts, 25 workgroups in the last, partly filled group
    (4, 8, 2, 128, 4100, dict(bit_set=(1, 2, 3, 4, 8)), False),                   # 16 parts: the plain order
    (8, 12, 2, 128, 1500, {}, False),                                             # 5 parts of 6 tiles
    (8, 4, 6, 128, 1500, {}, True),                            # four query heads per pass, and two left over: a tile per part
    (3, 7, 5, 64, 2600, {}, True),                             # ... one left over
    (16, 8, 8, 128, 1100, {}, True),                           # ... 3 parts, two workgroups per KV head
    (5, 3, 12, 64, 4700, {}, True),                            # ... 17 parts, three, 21 workgroups left over
    (4, 4, 8, 128, 5000, {}, True),                            # ... a tile per part
    (2, 2, 4, 128, 900, {}, False),                            # one kernel
])
def test_every_head_and_part_once(B, Hkv, G, D, T, kw, passes):
    print(f"shared codes: B={B} Hkv={Hkv} G={G} D={D} T={T} {kw}", flush=True)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(T + G)
    k, v = (torch.randn((B, Hkv, T, D), device="cuda", generator=gen).half() for _ in range(2))
    q = torch.randn((B, Hkv * G, D), device="cuda", generator=gen).half()
    c = qaq.Cache(qaq.make_config(B, Hkv * G, Hkv, D, T, [1.0] * Hkv, **kw))
    widths = torch.tensor(kw.get("bit_set", (2, 3, 4, 8)), dtype=torch.uint8, device="cuda")
    bits = [widths[torch.randint(len(widths), (B, Hkv, T), device="cuda", generator=gen)] for _ in range(2)]
    c.quantize_append(k, v, *bits)
    assert (attention_route(c).heads_per_scan == 4) == passes
    x, s = c.decode_attention(q, want_scores=True)
    kd, vd = (t.double() for t in c.dequantize())
    ref_s = ((q.double().view(B, Hkv, G, 1, D) * kd[:, :, None]).sum(-1) * D ** -0.5).softmax(-1)
    ref_x = (ref_s[..., None] * vd[:, :, None]).sum(-2).view(B, Hkv * G, D)
    ref_s = ref_s.view(B, Hkv * G, T)
    err_s = ((s - ref_s).abs().amax(-1) / ref_s.amax(-1)).max().item()
    err_x = ((x - ref_x).abs().amax(-1) / ref_x.abs().amax(-1)).max().item()
    print(f"  worst errors: scores {err_s:.1e}, output {err_x:.1e}", flush=True)
    assert err_s < TOL and err_x < TOL


@pytest.mark.parametrize("B,Hkv,G,D,T", [
    (9, 29, 1, 64, 513), (10, 32, 1, 128, 700), (31, 11, 1, 64, 1024), (5, 29, 2, 128, 2048), (10, 32, 1, 64, 2049), (19, 17, 1, 128, 2400)])
def test_a_little_more_heads_than_the_chip_has_units(B, Hkv, G, D, T):
    """257 to 341 heads: three parts a head are not in flight at once in one kernel, but are in two."""
    test_every_head_and_part_once(B, Hkv, G, D, T, {}, False)
