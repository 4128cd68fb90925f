"""Host-side checks that need no GPU: the library loads, exports what the header
declares, rejects bad arguments, and its code layout is a bijection."""
import ctypes as C
import os
import re

import numpy as np
import pytest

from paper_2403_04643_amd import qaq

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def _declared():
    """Every function declared in include/*.h (the product interface and the measurement / test aids)."""
    inc = os.path.join(ROOT, "include")
    names = set()
    for f in sorted(os.listdir(inc)):
        if f.endswith(".h"):
            text = re.sub(r"/\*.*?\*/", "", open(os.path.join(inc, f)).read(), flags=re.S)
            names |= set(re.findall(r"\b(qaq_[a-z0-9_]+)\s*\(", text))
    return sorted(names)


def test_library_exports_every_declared_symbol():
    lib = qaq.load()
    names = _declared()
    assert {"qaq_select_bits", "qaq_quantize_append", "qaq_requantize", "qaq_decode_attention",
            "qaq_dequantize"} <= set(names)
    for n in names:
        assert hasattr(lib, n), n
        assert n in qaq.SIGNATURES, f"binding lacks {n}"
    assert sorted(qaq.SIGNATURES) == names


def test_config_validation_without_gpu():
    lib = qaq.load()
    good = qaq.make_config(2, 8, 8, 128, 1000, [0.01] * 8)
    n = lib.qaq_arena_bytes(C.byref(good))
    assert n > 2 * 2 * 8 * 1024 * 128          # at least the 8-bit codes of K and V
    assert lib.qaq_outliers_per_side(C.byref(good)) == 1
    assert lib.qaq_arena_bytes(C.byref(qaq.make_config(2, 8, 8, 128, 1000, [0.01] * 8, bit_set=(1, 2, 3, 4, 8)))) == n
    for kw in (dict(head_dim=96), dict(bit_set=(2, 5)), dict(bit_set=(0, 2)), dict(bit_set=(3, 2)), dict(window=0),
               dict(n_outlier_per_side=5), dict(sigma_s_max=0.0), dict(n_q_heads=7)):
        args = dict(batch=2, n_q_heads=8, n_kv_heads=8, head_dim=128, max_tokens=1000, qnorm2=[0.01] * 8)
        args.update(kw)
        bad = qaq.make_config(**args)
        assert lib.qaq_arena_bytes(C.byref(bad)) == 0
        assert lib.qaq_last_error()
    h = C.c_void_p()
    assert lib.qaq_create(C.byref(good), None, n, C.byref(h)) == qaq.ERR_INVALID_ARG
    assert lib.qaq_create(C.byref(good), 256, n - 1, C.byref(h)) == qaq.ERR_CAPACITY
    assert lib.qaq_create(C.byref(good), 257, n, C.byref(h)) == qaq.ERR_INVALID_ARG
    assert lib.qaq_reset(None) == qaq.ERR_INVALID_ARG
    assert b"NULL" in lib.qaq_last_error()
    no_out = qaq.make_config(1, 4, 4, 64, 10, [1.0] * 4, outlier_frac=0.0)
    assert lib.qaq_outliers_per_side(C.byref(no_out)) == 0
    four = qaq.make_config(1, 4, 4, 128, 10, [1.0] * 4, outlier_frac=0.05)
    assert lib.qaq_outliers_per_side(C.byref(four)) == 4


@pytest.mark.parametrize("side", [0, 1])
@pytest.mark.parametrize("D", [64, 128])
def test_layout_is_a_bijection(side, D):
    """Every code bit of every token lands on its own bit of the tile image, inside the
    region bounds and the reserved capacity; the image has no other holes than the
    documented padding."""
    rng = np.random.default_rng(D + side)
    cap = qaq.load().qaq_debug_tile_capacity(side, D)
    cases = [(256, 0, 0, 0, 0), (0, 256, 0, 0, 0), (0, 0, 256, 0, 0), (0, 0, 0, 256, 0), (0, 0, 0, 0, 256),
             (1, 1, 1, 1, 1), (17, 9, 3, 33, 21), (1, 1, 1, 252, 1)]
    for k in range(6):
        cut = np.sort(rng.integers(0, 257, 4))
        if k < 3:
            cut[3] = 256                      # no 1-bit tokens: the layout of the paper's width set
        cases.append((cut[0], cut[1] - cut[0], cut[2] - cut[1], cut[3] - cut[2], 256 - cut[3]))
    for n3, n2, n4, n8, n1 in cases:
        counts = (int(n3), int(n2), int(n4), int(n8), int(n1))
        used = np.zeros(cap * 8, dtype=np.uint8)
        end = None
        def mark(bf, idx, width_mask_bits):
            nonlocal end
            for d in range(D):
                off, sh, end = qaq.debug_field(side, D, counts, bf, idx, d)
                assert off % 4 == 0 and sh + width_mask_bits <= 32
                lo = off * 8 + sh
                assert lo + width_mask_bits <= end * 8 <= cap * 8
                assert not used[lo:lo + width_mask_bits].any(), (counts, bf, idx, d)
                used[lo:lo + width_mask_bits] = 1
        for s in range(n3 + n2):
            mark(2, s, 2)
        for s in range(n3):
            mark(1, s, 1)
        for s in range(n4):
            mark(4, s, 4)
        for s in range(n8):
            mark(8, s, 8)
        for s in range(n1):
            mark(0, s, 1)
        total_bits = D * (3 * n3 + 2 * n2 + 4 * n4 + 8 * n8 + n1)
        assert used.sum() == total_bits
        if end is not None:
            pad = end * 8 - total_bits
            # at most one partly filled group per region: keys 15 records of D/4 + D/8 + D/2 + D/8
            # bytes, values 15/16 of a 4D- and of two 2D-byte units and 7/8 of a 4D-byte half-unit
            assert pad <= 8 * (15 * D)


def test_stream_lookup_keeps_torchs_checks(monkeypatch):
    """The current stream's handle is asked for past the object around it, but not past what torch refuses (a process forked
    after the GPU's first use), and by the public way where the private one is not there."""
    torch = pytest.importorskip("torch")
    monkeypatch.setattr(torch.cuda, "_is_in_bad_fork", lambda: True)
    with pytest.raises(RuntimeError, match="fork"):
        qaq._stream()
    monkeypatch.delattr(torch._C, "_cuda_getCurrentRawStream")
    monkeypatch.setattr(torch.cuda, "current_stream", lambda: type("Stream", (), {"cuda_stream": 7}))
    assert qaq._stream() == 7


@pytest.mark.parametrize("D", [64, 128])
def test_attention_route_covers_every_tile(D):
    """However a call goes: parts that hold all tiles, none of them more than a workgroup's tables, and no more parts than the
    cache's arena has places for."""
    for B, Hkv, G in ((1, 1, 1), (1, 8, 1), (10, 32, 1), (16, 32, 1), (40, 32, 1), (16, 8, 2), (1, 8, 3), (16, 8, 3), (48, 8, 3),
                      (1, 8, 4), (8, 8, 4), (16, 8, 5), (16, 8, 7), (16, 8, 8), (16, 8, 9), (64, 32, 4)):
        for n_o, bit_set in ((-1, (2, 3, 4, 8)), (0, (2, 3, 4, 8)), (3, (2, 3, 4, 8)), (-1, (1, 2, 3, 4, 8))):
            cfg = qaq.make_config(B, Hkv * G, Hkv, D, 65536, [1.0] * Hkv, bit_set=bit_set, n_outlier_per_side=n_o)
            for T in (1, 256, 257, 700, 1500, 4096, 33000, 65536):
                for shortest in (T, (T + 1) // 2, 0):
                    r = qaq.attention_route(cfg, T, shortest)
                    tiles = (T + 255) // 256
                    assert 1 <= r.parts <= tiles and r.parts * r.tiles >= tiles and r.parts * (r.tiles - 1) < tiles and r.tiles <= 64
                    assert r.heads_per_scan == 1 or (G > 2 and n_o < 1 and bit_set[0] == 2)
                    assert r.kernels == 1 or r.kernels == 2
                    if r.kernels == 1:      # the parts are one workgroup and every one has a tile, and nothing is left to merge
                        assert r.heads_per_scan == 1 and r.parts <= 4 and (shortest == T or (shortest + 255) // 256 >= r.parts) and r.static_bytes == 0
    empty = qaq.attention_route(cfg, 0)
    assert empty.kernels == 0
    with pytest.raises(qaq.QaqError):
        qaq.attention_route(cfg, 65537)


@pytest.mark.parametrize("G", [4, 8, 12])
def test_full_groups_have_parts_as_short_as_in_passes_of_four(G):
    """The rounding error of an output grows with the tiles of a part, so a call that could go in passes of four query heads --
    three workgroups per compute unit -- has no longer parts where it goes in a scan per head."""
    routes = set()
    for B in list(range(1, 20)) + [24, 32, 48, 64]:
        for Hkv in (1, 2, 8, 16, 32):
            cfg = qaq.make_config(B, Hkv * G, Hkv, 128, 16384, [1.0] * Hkv)
            for T in (1, 250, 256, 257, 500, 700, 1000, 1025, 1500, 2000, 3000, 5000, 16384):
                tiles = (T + 255) // 256
                parts = min(tiles, max(1, 3 * 256 // (B * Hkv * G // 4)))
                for shortest in (T, T // 2 + 1):
                    r = qaq.attention_route(cfg, T, shortest)
                    assert r.tiles <= -(-tiles // parts), (B, Hkv, T, shortest)
                    routes.add((r.heads_per_scan, r.kernels))
    assert routes == {(1, 1), (1, 2), (4, 2)}


@pytest.mark.parametrize("B,Hkv,G,T,passes,parts", [
    (24, 8, 5, 600, False, 1), (12, 8, 5, 616, False, 2), (16, 16, 3, 500, False, 1),       # where a scan per head is faster
    (32, 8, 3, 700, True, 3), (14, 8, 9, 979, True, 2), (24, 4, 7, 1785, True, 4), (22, 16, 3, 1030, True, 2), (16, 8, 7, 8192, True, 3),
    (16, 8, 3, 8192, True, 6), (21, 8, 3, 1476, False, 2), (47, 1, 11, 1286, True, 3), (19, 32, 5, 356, True, 1), (4, 8, 5, 7032, True, 12)])
def test_groups_that_are_not_full_have_the_parts_the_chip_holds(B, Hkv, G, T, passes, parts):
    """... and go in passes of four only where those are the faster ones."""
    r = qaq.attention_route(qaq.make_config(B, Hkv * G, Hkv, 128, T, [1.0] * Hkv), T)
    assert (r.heads_per_scan == 4, r.parts) == (passes, parts)


@pytest.mark.parametrize("D", [64, 128])
def test_static_calls_that_keep_off_the_shared_array(D):
    """Two qaq_decode_attention_static calls on two caches may overlap where neither uses the library's array: all calls whose
    heads are at most four workgroups each, except where the passes of four query heads fill their four."""
    seen = set()
    for B, Hkv, G in ((1, 1, 1), (9, 32, 1), (10, 32, 1), (341, 1, 1), (10, 16, 2), (16, 8, 2), (16, 8, 3), (48, 8, 3), (16, 8, 5), (8, 8, 7),
                      (16, 8, 7), (16, 8, 9), (14, 8, 11), (40, 32, 1), (1, 8, 5)):
        for T in (100, 700, 1300, 2000, 4096, 8192):
            cfg = qaq.make_config(B, Hkv * G, Hkv, D, T, [1.0] * Hkv)
            tiles = (T + 255) // 256
            a_head = min(tiles, max(1, 4 * 256 // (B * Hkv * G)))
            for scores in (False, True):
                r = qaq.attention_route(cfg, T, with_scores=scores)
                alone = a_head <= 4 and (a_head == 4 or a_head * -(-tiles // a_head) <= 32 or not scores)      # (raw logits in LDS)
                assert (r.static_bytes == 0) == alone, (B, Hkv, G, T, scores)
                assert r.static_bytes <= qaq.load().qaq_static_scratch_limit()
                seen.add((alone, r.kernels, r.heads_per_scan))
    assert {(True, 1, 1), (True, 2, 1), (True, 2, 4), (False, 2, 1), (False, 2, 4)} <= seen


# ---- code objects in the built library: the kernels on the decode path keep their working set in registers ----

def _gfx950_code_objects(path):
    """The gfx950 code objects inside the library's .hip_fatbin section (one offload bundle per source file;
    bundle layout: magic, u64 entry count, then per entry u64 offset, u64 size, u64 triple length, triple)."""
    import struct
    import subprocess
    import tempfile
    objcopy = "/opt/rocm/llvm/bin/llvm-objcopy"
    if not os.path.exists(objcopy):
        pytest.skip("llvm-objcopy not found")
    with tempfile.TemporaryDirectory() as d:
        fat = os.path.join(d, "fat.bin")
        subprocess.run([objcopy, f"--dump-section=.hip_fatbin={fat}", path, os.path.join(d, "unused")], check=True)
        blob = open(fat, "rb").read()
    magic = b"__CLANG_OFFLOAD_BUNDLE__"
    out = []
    at = blob.find(magic)
    while at >= 0:
        p = at + len(magic)
        (n,) = struct.unpack_from("<Q", blob, p)
        p += 8
        for _ in range(n):
            off, size, tl = struct.unpack_from("<QQQ", blob, p)
            triple = blob[p + 24:p + 24 + tl].decode()
            p += 24 + tl
            if "gfx950" in triple:
                out.append(blob[at + off:at + off + size])
        at = blob.find(magic, at + len(magic))
    return out


def _kernel_metadata(code_object):
    """name -> metadata map of every kernel of one code object (the msgpack document of the NT_AMDGPU_METADATA note)."""
    import struct
    import msgpack
    e = code_object
    assert e[:4] == b"\x7fELF" and e[4] == 2
    shoff, = struct.unpack_from("<Q", e, 0x28)
    shentsize, shnum = struct.unpack_from("<HH", e, 0x3A)
    kernels = {}
    for i in range(shnum):
        sh = shoff + i * shentsize
        sh_type, = struct.unpack_from("<I", e, sh + 4)
        off, size = struct.unpack_from("<QQ", e, sh + 0x18)
        if sh_type != 7:       # SHT_NOTE
            continue
        p = off
        while p + 12 <= off + size:
            namesz, descsz, ntype = struct.unpack_from("<III", e, p)
            name = e[p + 12:p + 12 + namesz]
            desc_at = p + 12 + ((namesz + 3) & ~3)
            if name.rstrip(b"\0") == b"AMDGPU" and ntype == 32:
                doc = msgpack.unpackb(e[desc_at:desc_at + descsz], raw=False, strict_map_key=False)
                for k in doc.get("amdhsa.kernels", []):
                    kernels[k[".name"]] = k
            p = desc_at + ((descsz + 3) & ~3)
    return kernels


def test_decode_path_kernels_do_not_spill():
    """A change elsewhere in a source file can push a kernel over its register budget or make the compiler call
    its helpers out of line; both show as private (scratch) memory in the kernel's metadata long before a test of
    the results notices anything.  The kernels of a decode step and of the bulk quantization at the benchmark's
    shape (head_dim 128, one outlier per end, no 1-bit width) are held to none."""
    if not os.path.exists(qaq.LIB_PATH):
        pytest.skip("library not built")
    kernels = {}
    for co in _gfx950_code_objects(qaq.LIB_PATH):
        kernels.update(_kernel_metadata(co))
    assert kernels, "no gfx950 code object found in the library"
    held = {"k_attn_tileILi128ELi2ELi4ELb0": 128, "k_attn_tileILi128ELi2ELi0ELb0": 128, "k_updateILi128": 64,
            "k_selectE": 128, "k_buildILi128ELb1ELb0": 128, "k_attn_combineILi128": 128}
    seen = set()
    for name, k in kernels.items():
        for key, max_vgpr in held.items():
            if key in name:
                seen.add(key)
                assert k[".private_segment_fixed_size"] == 0, (name, k[".private_segment_fixed_size"])
                assert k[".vgpr_count"] <= max_vgpr, (name, k[".vgpr_count"])
    assert seen == set(held), set(held) - seen


@pytest.mark.parametrize("key,max_vgpr,max_scratch", [
    ("k_attn_tileILi128ELi8E", 128, 48),      # several outliers per end: a few words spilled, and no more
    ("k_attn_tileILi64ELi8E", 128, 0),
    ("k_attn_tileILi128ELi16E", 128, 72),     # outliers by thresholds
    ("k_attn_tileILi64ELi16E", 128, 20),
    ("k_build_listedILi128ELb1E", 128, 0),    # four, three, five and four workgroups per compute unit, as the launch counts on
    ("k_build_listedILi128ELb0E", 168, 0),
    ("k_build_listedILi64ELb1E", 96, 0),
    ("k_build_listedILi64ELb0E", 128, 0),
    ("k_buildILi128ELb1E", 128, 0),           # four, three, seven and four wavefronts per SIMD
    ("k_buildILi128ELb0E", 168, 0),
    ("k_buildILi64ELb1E", 72, 0),
    ("k_buildILi64ELb0E", 128, 0),
    ("k_attn_gqaILi128ELi2E", 168, 0),        # three workgroups per compute unit
    ("k_attn_gqaILi128ELi0E", 168, 0),
    ("k_attn_gqaILi64E", 168, 0),
    ("k_dequantILi128ELi2E", 64, 0),          # eight wavefronts per SIMD
    ("k_dequantILi128ELi0E", 64, 0),
    ("k_dequantILi64ELi2E", 64, 0),
    ("k_dequantILi64ELi0E", 64, 0),
    ("k_dequantILi128ELi8E", 72, 0),          # seven
    ("k_dequantILi64ELi8E", 72, 0),
    ("k_update_fewI", 64, 0),                 # eight (scalar registers: six)
    ("k_prefill_softmaxILi64E", 256, 0),      # 64 logits per thread
    ("k_prefill_softmax_wideILi8E", 64, 0),   # two rows of sixteen wavefronts per compute unit
    ("k_prefill_softmax_wideILi16E", 64, 0),
    ("k_prefill_softmax_wideILi20E", 64, 0),
    ("k_prefill_softmax_wideILi32E", 128, 0), # one
])
def test_other_kernels_at_their_budget(key, max_vgpr, max_scratch):
    """The same for kernels off the benchmark's shape that sit at the edge of their budget: one register more in each
    lane there was 10 % of an attention call."""
    if not os.path.exists(qaq.LIB_PATH):
        pytest.skip("library not built")
    found = 0
    for co in _gfx950_code_objects(qaq.LIB_PATH):
        for name, k in _kernel_metadata(co).items():
            if key in name:
                found += 1
                assert k[".private_segment_fixed_size"] <= max_scratch, (name, k[".private_segment_fixed_size"])
                assert k[".vgpr_count"] <= max_vgpr, (name, k[".vgpr_count"])
    assert found, key


def test_the_steps_calls_pass_what_they_are_given():
    """_qaq_call: addresses of tensors, of page-locked buffers and of nothing, the stream, the output's type and the status, in
    the order of the C functions; what the binding refuses, refused."""
    if not os.path.exists(qaq.LIB_PATH):
        pytest.skip("library not built")
    torch = pytest.importorskip("torch")
    import ctypes as C
    call = qaq._load_call()

    class Tensor:
        is_cuda, dtype = True, torch.float32

        def __init__(self, at, contiguous=True):
            self.at, self.contiguous = at, contiguous

        def is_contiguous(self):
            return self.contiguous

        def data_ptr(self):
            return self.at

    got = []
    vp, i32 = C.c_void_p, C.c_int32
    fn_a = C.CFUNCTYPE(C.c_int, vp, vp, vp, vp, vp, i32, vp, vp)(lambda *a: got.append(a) or -3)
    fn_u = C.CFUNCTYPE(C.c_int, vp, vp, vp, vp, vp, vp, i32, vp, vp, vp)(lambda *a: got.append(a) or 0)
    at_a, at_u = (C.cast(f, vp).value for f in (fn_a, fn_u))
    buf = qaq.HostBuffer.__new__(qaq.HostBuffer)
    buf.dev_ptr = 0xB0F
    big = 0x7fff_ffff_fff0
    try:
        call.setup(qaq.HostBuffer, torch.float32, lambda: 3, lambda dev: 0x500 + dev, None)
        assert call.attention(at_a, big, Tensor(1), None, None, Tensor(2), Tensor(big)) == -3
        assert got.pop() == (big, 1, None, None, 2, 1, big, 0x503)
        half = Tensor(2)
        half.dtype = torch.float16
        call.attention(at_a, big, Tensor(1), Tensor(7), Tensor(8), half, None)
        assert got.pop() == (big, 1, 7, 8, 2, 0, None, 0x503)
        call.setup(qaq.HostBuffer, torch.float32, None, None, lambda: 0)      # torch without those lookups
        assert call.update(at_u, 5, Tensor(1), Tensor(2), Tensor(3), buf, None, 77, None, Tensor(4)) == 0
        assert got.pop() == (5, 1, 2, 3, 0xB0F, None, 77, None, 4, None)
        for bad in (Tensor(1, contiguous=False), torch.zeros(2)):
            with pytest.raises(AssertionError, match="contiguous CUDA tensors"):
                call.attention(at_a, big, bad, None, None, Tensor(2), None)
        for bad in (3, "q"):
            with pytest.raises(AttributeError):
                call.update(at_u, 5, Tensor(1), Tensor(2), Tensor(3), bad, None, 77, None, None)
        with pytest.raises(TypeError):
            call.attention(at_a, big, Tensor(1))
        assert not got
    finally:
        buf.__dict__.clear()
        qaq._call = None
        qaq._load_call()


def test_the_extension_is_for_this_python():
    """It is built against one Python's headers: its name tells the others to leave it alone."""
    if not os.path.exists(qaq.LIB_PATH):
        pytest.skip("library not built")
    pytest.importorskip("torch")
    import sysconfig
    assert sysconfig.get_config_var("SOABI") and os.path.basename(qaq._load_call().__file__) == "_qaq_call" + sysconfig.get_config_var("EXT_SUFFIX")


def test_what_needs_no_cache_needs_neither_torch_nor_the_extension():
    """Sizes, limits and routes by ctypes alone; a cache without the extension says how to build it."""
    if not os.path.exists(qaq.LIB_PATH):
        pytest.skip("library not built")
    import subprocess
    import sys
    code = '''
import ctypes as C, sys
sys.modules["paper_2403_04643_amd._qaq_call"] = None
%s
from paper_2403_04643_amd import qaq
cfg = qaq.make_config(2, 8, 8, 128, 1000, [0.01] * 8)
assert qaq.load().qaq_arena_bytes(C.byref(cfg)) > 0 and qaq.attention_route(cfg, 1000).parts > 0
try:
    qaq.Cache(cfg)
except %s as e:
    assert %r in str(e), e
else:
    raise SystemExit("a cache without what it needs")
'''
    for block, error, says in (('sys.modules["torch"] = None', "ImportError", "torch"), ("", "RuntimeError", "build it with")):
        r = subprocess.run([sys.executable, "-c", code % (block, error, says)], cwd=ROOT, capture_output=True, text=True, timeout=300)
        assert r.returncode == 0, r.stderr
