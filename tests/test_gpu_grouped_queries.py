"""Grouped-query attention (four query heads per pass over the codes) where its kernel divides a tile: a wavefront takes every
fourth group of 16 key slots, eight 8-bit keys and values per wavefront and sixteen 4-bit values come with the tile, weight
tables reach as far as blocks of 64 slots do."""
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from paper_2403_04643_amd import qaq  # noqa: E402
from tests.parity_util import attention_route  # noqa: E402

def stored(c, side):
    """Per sequence its stored tokens in 64 bits (behind the end of a shorter one the export writes nothing: no index there is
    one).  A code is where the fp16 reconstruction lies (2^-11 of a value at most half a segment, 2^-9 of the range: the
    token's largest value is below twice its range)."""
    e, xs = c.export_canonical(side), c.dequantize()[side]
    out = []
    for b, m in enumerate(c.lengths()):
        mn, mx = (t[..., None] for t in e["minmax"][b, :, :m].double().unbind(-1))
        seg = (mx - mn) * torch.exp2(-e["bits"][b, :, :m].double())[..., None]
        x = mn + (((xs[b, :, :m].double() - mn) / seg - 0.5).round() + 0.5) * seg
        out.append(x.scatter_(-1, e["oidx"][b, :, :m].long(), e["oval"][b, :, :m].double()))
    return out


def check(c, q, x, s):
    """Outputs and scores against 64 bits over what is stored, for K, V and queries within +-4.  Scores: the query's 22 bits
    leave at most 128 * 2^-23 * 4 * 8 / sqrt(128) in a logit, twice that in a score; 32-bit sums add a few 1e-6."""
    kd, vd = stored(c, 0), stored(c, 1)
    Hkv, G, D = c.cfg.n_kv_heads, c.cfg.n_q_heads // c.cfg.n_kv_heads, c.cfg.head_dim
    for b, m in enumerate(c.lengths()):
        p = (torch.matmul(q[b].double().view(Hkv, G, D), kd[b].transpose(-1, -2).contiguous()) * D ** -0.5).softmax(-1)
        ref = torch.matmul(p, vd[b])
        got = s[b, :, :m].double().view(Hkv, G, m)
        assert ((got - p).abs().amax(-1) / p.amax(-1)).max().item() < 2e-4
        assert ((x[b].double().view(Hkv, G, D) - ref).abs().amax(-1) / ref.abs().amax(-1)).max().item() < 4e-4


@pytest.mark.parametrize("counts", [       # 3, 2, 4, 8 bits in the last tile
    (0, 1, 0, 0), (1, 0, 0, 0), (0, 0, 1, 0), (0, 0, 0, 1), (15, 1, 0, 0), (16, 0, 0, 1), (17, 14, 1, 1),
    (64, 150, 12, 9), (65, 127, 16, 8), (63, 160, 17, 16), (129, 100, 18, 9), (128, 0, 64, 64), (0, 191, 65, 0),
    (0, 240, 0, 16), (0, 247, 0, 9), (200, 0, 30, 26), (256, 0, 0, 0), (0, 256, 0, 0), (0, 0, 256, 0), (0, 0, 0, 256), (3, 250, 2, 1)])
@pytest.mark.parametrize("D,n_o", [(128, 1), (64, 1), (128, 0)])
def test_class_borders(counts, D, n_o):
    """Full groups, a part per tile: four tiles with the last one's classes at other borders, then that one."""
    n = sum(counts)
    B, Hkv, G, T = 4, 8, 4, 1024 + n
    print(f"class borders: {counts} D={D} n_o={n_o}", flush=True)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(1000 * counts[0] + counts[1] + D + n_o)
    k, v = (torch.randn((B, Hkv, T, D), device="cuda", generator=gen).clamp_(-4, 4).half() for _ in range(2))
    q = torch.randn((B, Hkv * G, D), device="cuda", generator=gen).clamp_(-4, 4).half()
    c = qaq.Cache(qaq.make_config(B, Hkv * G, Hkv, D, T, [1.0] * Hkv, n_outlier_per_side=n_o))

    def widths(cn):
        w = torch.tensor(sum(([b] * m for b, m in zip((3, 2, 4, 8), cn)), []), dtype=torch.uint8, device="cuda")
        return torch.stack([w[torch.randperm(len(w), device="cuda", generator=gen)] for _ in range(B * Hkv)]).view(B, Hkv, -1)

    first = (256 - n + counts[0],) + counts[1:]
    c.quantize_append(k, v, *(torch.cat([widths(first) for _ in range(4)] + [widths(counts)], dim=2).contiguous() for _ in range(2)))
    assert attention_route(c).heads_per_scan == 4
    x, s = c.decode_attention(q, want_scores=True)
    check(c, q, x, s)


@pytest.mark.parametrize("D", [128, 64])
@pytest.mark.parametrize("B,G,T", [(16, 4, 1280), (25, 3, 1280), (1, 4, 512), (1, 1, 512)])      # passes of four, full and not; scans
@pytest.mark.parametrize("value", [1.99, -1.99, 1.0])
def test_one_channel_carries_everything(D, B, G, T, value):
    """The largest sums an outlier correction can have: equal weights (a query of zeros) over full tiles of tokens whose one
    channel that is not zero has a value just below a power of two."""
    Hkv = 2
    c = qaq.Cache(qaq.make_config(B, Hkv * G, Hkv, D, T, [1.0] * Hkv, n_outlier_per_side=1))
    v = torch.zeros((B, Hkv, T, D), dtype=torch.float16, device="cuda")
    v[..., 7] = value
    k = torch.randn((B, Hkv, T, D), device="cuda", generator=torch.Generator(device="cuda").manual_seed(D + G)).half()
    two = torch.full((B, Hkv, T), 2, dtype=torch.uint8, device="cuda")
    c.quantize_append(k, v, two, two)
    assert attention_route(c, with_scores=False).heads_per_scan == (4 if B > 1 else 1)
    x, _ = c.decode_attention(torch.zeros((B, Hkv * G, D), dtype=torch.float16, device="cuda"))
    want = v[:, :, :1].float().expand(B, Hkv, G, D).reshape(B, Hkv * G, D)
    # every correction is off by at most half a unit of 2^-25 of the bound, the sums by a few roundings of 32 bits
    assert (x - want).abs().max().item() < 4e-6


@pytest.mark.parametrize("counts", [       # 3, 2, 4, 8 bits in the last tile
    (0, 1, 0, 0), (17, 14, 1, 1), (65, 127, 16, 8), (63, 160, 17, 16), (128, 0, 64, 64), (0, 0, 0, 256), (3, 250, 2, 1)])
@pytest.mark.parametrize("B,Hkv,G,D,n_o,tiles", [
    (48, 8, 3, 128, 1, 2), (48, 8, 3, 64, 0, 2), (32, 8, 5, 128, 1, 2), (32, 8, 5, 128, 0, 2), (24, 8, 7, 64, 1, 2), (24, 8, 6, 128, 1, 2),
    (32, 8, 4, 128, 1, 2), (32, 8, 4, 128, 0, 2), (16, 8, 8, 64, 1, 2), (4, 8, 5, 128, 1, 16), (2, 8, 3, 64, 1, 33)])
def test_groups_that_are_not_full(counts, B, Hkv, G, D, n_o, tiles):
    """Caches large enough for four heads per pass, the last pass of a group with one, two, three and four heads; the longer ones
    with sequences too short for every part to have a tile."""
    n = sum(counts)
    T, Hq = 256 * (tiles - 1) + n, Hkv * G
    short = [0] * B if tiles == 2 else [(T - 300) * (b % 2) for b in range(B)]
    print(f"groups: {counts} B={B} Hkv={Hkv} G={G} D={D} n_o={n_o} T={T}", flush=True)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(1000 * counts[0] + counts[1] + D + G)
    k, v = (torch.randn((B, Hkv, T, D), device="cuda", generator=gen).clamp_(-4, 4).half() for _ in range(2))
    q = torch.randn((B, Hq, D), device="cuda", generator=gen).clamp_(-4, 4).half()
    c = qaq.Cache(qaq.make_config(B, Hq, Hkv, D, T, [1.0] * Hkv, n_outlier_per_side=n_o))
    if any(short):
        c.set_shortfall(short)
    last = torch.tensor(sum(([w] * m for w, m in zip((3, 2, 4, 8), counts)), []), dtype=torch.uint8, device="cuda")
    bits = []
    for _ in range(2):
        w = torch.tensor((2, 2, 2, 3, 3, 4, 8), dtype=torch.uint8, device="cuda")[torch.randint(7, (B, Hkv, T), device="cuda", generator=gen)]
        w[:, :, T - n:] = last[torch.rand((B, Hkv, n), device="cuda", generator=gen).argsort(dim=-1)]
        bits.append(w.contiguous())
    c.quantize_append(k, v, *bits)
    assert attention_route(c).heads_per_scan == 4
    c.profile_begin(1)
    s = torch.zeros((B, Hq, T), device="cuda")
    x, _ = c.decode_attention(q, scores_out=s)
    assert c.profile_read()[1][0] > 0.0          # a merge kernel
    out = torch.full((B, Hq, D), float("nan"), device="cuda")
    if G % 4 != 0:                               # (full groups may exceed the static scratch)
        c.decode_attention_static(q, None, None, out)
        assert torch.equal(out, x)
    check(c, q, x, s)
