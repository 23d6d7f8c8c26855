"""Host-side checks that need no GPU: the library loads, exports every symbol the header declares,
and validates its arguments before touching the device."""
import ctypes
import os
import re

import numpy as np
import pytest

from tests import helpers as Hp

from paper_2604_10496_amd import binding as B, synth

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def _declared_functions():
    found = set()
    for header in ("cq.h", "cq_measure.h"):
        text = open(os.path.join(ROOT, "include", header)).read()
        text = re.sub(r"/\*.*?\*/", "", text, flags=re.S)
        found |= set(re.findall(r"\b(cq_[a-z0-9_]+)\s*\(", text))
    return sorted(found)


def test_header_and_library_agree():
    if not os.path.exists(B.LIB_PATH):
        pytest.fail("libcq.so is not built: run `python -m paper_2604_10496_amd.build`")
    lib = B.load_library()
    declared = _declared_functions()
    assert len(declared) >= 14
    for name in declared:
        assert hasattr(lib, name), f"{name} is declared in cq.h but not exported"
    assert sorted(B.EXPORTS) == declared


def test_status_strings():
    lib = B.load_library()
    seen = {lib.cq_status_string(i) for i in range(6)}
    assert len(seen) == 6 and lib.cq_status_string(0) == b"CQ_OK"


def test_argument_validation_happens_before_any_device_call():
    lib = B.load_library()
    one = ctypes.c_void_p(256)   # a non-null dummy that must never be dereferenced
    # rotate_quant
    assert lib.cq_rotate_quant(None, one, 4, 64, 8, one, one, one, one, 1 << 20, None) == 1
    assert lib.cq_rotate_quant(one, one, 0, 64, 8, one, one, one, one, 1 << 20, None) == 2
    assert lib.cq_rotate_quant(one, one, 4, 100, 8, one, one, one, one, 1 << 20, None) == 2
    assert lib.cq_rotate_quant(one, one, 4, 64, 5, one, one, one, one, 1 << 20, None) == 3
    assert lib.cq_rotate_quant(one, one, 16, 4096, 8, one, one, one, None, 0, None) == 4
    # route_permute
    args = lambda **k: [k.get("XR", one), one, None, None, k.get("T", 8), 64, k.get("E", 8), k.get("k", 2), 0,
                        None, one, one, one, one, one, None, k.get("ws", one), k.get("wsb", 1 << 24), None]
    assert lib.cq_route_permute(*args(k=9)) == 2
    assert lib.cq_route_permute(*args(E=2000)) == 2
    assert lib.cq_route_permute(*args(XR=None)) == 1
    assert lib.cq_route_permute(*args(wsb=8)) == 4
    # grouped gemm
    W = B.CodebookWeights(256, 256, None, 2, 128, 128)
    g = lambda W, a_kind=0, epi=0, outk=0: lib.cq_codebook_grouped_gemm(ctypes.byref(W), one, a_kind, None, None,
                                                                        one, 4, epi, one, outk, None, 0, None)
    assert g(B.CodebookWeights(None, 256, None, 2, 128, 128)) == 1
    assert g(B.CodebookWeights(256, 256, None, 2, 100, 128)) == 2
    assert g(B.CodebookWeights(256, 256, None, 2, 128, 96)) == 2
    assert g(W, a_kind=7) == 3 and g(W, epi=5) == 3 and g(W, outk=9) == 3
    # the lookup formulation of the product
    gl = lambda W, epi=0, outk=0, codes=one: lib.cq_codebook_grouped_gemm_lut(ctypes.byref(W), codes, None, None,
                                                                             one, 4, epi, one, outk, None)
    assert gl(W, codes=None) == 1
    assert gl(B.CodebookWeights(None, 256, 256, 2, 128, 128)) == 1          # canonical bytes are required
    assert gl(B.CodebookWeights(256, 256, None, 2, 100, 128)) == 2
    assert gl(B.CodebookWeights(256, 256, None, 2, 128, 128, 48)) == 2      # groups of 48 weights
    assert gl(W, epi=5) == 3 and gl(W, outk=9) == 3
    # block-wise tables in the matrix-core product: groups must be multiples of 512 weights, rows of 256
    assert g(B.CodebookWeights(256, 256, None, 2, 256, 1024, 256)) == 3
    assert g(B.CodebookWeights(256, 256, None, 2, 128, 1024, 512)) == 3
    assert g(B.CodebookWeights(256, 256, None, 2, 128, 1024, -4)) == 2
    # smaller centroid budgets
    ex = lambda bits=2, K=128, src=one: lib.cq_expand_centroid_budget(src, one, bits, 2, 64, K, 1, one, one, None)
    assert ex(src=None) == 1 and ex(K=100) == 2 and ex(bits=4) == 3 and ex(bits=1) == 3
    # moe_forward: shape mismatch between layer and weights, bad bits
    gu = B.CodebookWeights(256, 256, None, 4, 256, 128)
    dn = B.CodebookWeights(256, 256, None, 4, 128, 128)
    L = B.Layer(128, 128, 4, 2, 0, 8, 256, 256, None, gu, dn)
    assert lib.cq_moe_workspace_bytes(ctypes.byref(L), 16) > 0
    assert lib.cq_moe_forward(ctypes.byref(L), one, 16, one, None, 0, None) == 4
    # the entry point with the library's own scratch array: same validation, and a batch beyond the array's
    # size is refused before any device call
    assert lib.cq_moe_forward_static(ctypes.byref(L), None, 16, one, None) == 1
    assert lib.cq_moe_forward_static(ctypes.byref(L), one, 0, one, None) == 2
    assert lib.cq_moe_workspace_bytes(ctypes.byref(L), 1 << 16) > (32 << 20)
    assert lib.cq_moe_forward_static(ctypes.byref(L), one, 1 << 16, one, None) == 4
    Lbad = B.Layer(128, 128, 4, 2, 0, 6, 256, 256, None, gu, dn)
    assert lib.cq_moe_forward(ctypes.byref(Lbad), one, 16, one, one, 1 << 30, None) == 3
    Lbad2 = B.Layer(128, 128, 4, 5, 0, 8, 256, 256, None, gu, dn)
    assert lib.cq_moe_forward(ctypes.byref(Lbad2), one, 16, one, one, 1 << 30, None) == 2
    Lbad3 = B.Layer(128, 64, 4, 2, 0, 8, 256, 256, None, gu, dn)
    assert lib.cq_moe_forward(ctypes.byref(Lbad3), one, 16, one, one, 1 << 30, None) == 2
    # block-wise tables the kernels cannot take: refused for the layer as well
    gu_b = B.CodebookWeights(256, 256, None, 4, 256, 128, 64)
    Lblk = B.Layer(128, 128, 4, 2, 0, 8, 256, 256, None, gu_b, dn)
    assert lib.cq_moe_workspace_bytes(ctypes.byref(Lblk), 16) == 0
    assert lib.cq_moe_forward(ctypes.byref(Lblk), one, 16, one, one, 1 << 30, None) == 3
    # prepack / decode
    assert lib.cq_prepack(ctypes.byref(W), one, 8, None) == 4
    assert lib.cq_decode_dense(ctypes.byref(W), 5, one, None) == 2
    assert lib.cq_stream_read(one, 24, one, None) == 2
    assert lib.cq_mfma_loop(8, 10, None, None) == 1 and lib.cq_mfma_loop(0, 10, one, None) == 2
    # split copy of R and the rotation that uses it
    assert lib.cq_rotation_split_bytes(256) == 256 * 256 * 4 and lib.cq_rotation_split_bytes(100) == 0
    assert lib.cq_rotation_split(None, 256, one, 1 << 30, None) == 1
    assert lib.cq_rotation_split(one, 100, one, 1 << 30, None) == 2
    assert lib.cq_rotation_split(one, 256, one, 16, None) == 4
    assert lib.cq_rotate_quant_split(one, None, 256, 256, 8, one, one, one, one, 1 << 30, None) == 1
    assert lib.cq_rotate_quant_split(one, one, 100, 256, 8, one, one, one, one, 1 << 30, None) == 2   # too few tokens
    assert lib.cq_rotate_quant_split(one, one, 256, 192, 8, one, one, one, one, 1 << 30, None) == 2   # H % 256
    assert lib.cq_rotate_quant_split(one, one, 256, 256, 5, one, one, one, one, 1 << 30, None) == 3
    assert lib.cq_rotate_quant_split(one, one, 256, 256, 8, one, one, one, one, 64, None) == 4
    assert lib.cq_rotate_quant_split_workspace_bytes(256, 256) >= 2 * 256 * 256 * 2 + 256 * 4
    # online-Hadamard transform of rows
    assert lib.cq_hadamard_quant(None, 4, 512, 8, None, one, one, None) == 1
    assert lib.cq_hadamard_quant(one, 4, 320, 8, None, one, one, None) == 2       # 5 * 64: no such matrix here
    assert lib.cq_hadamard_quant(one, 4, 1 << 15, 8, None, one, one, None) == 2   # row longer than LDS holds
    assert lib.cq_hadamard_quant(one, 4, 768, 5, None, one, one, None) == 3
    assert lib.cq_hadamard_quant(None, 0, 768, 8, None, None, None, None) == 0


def test_workspace_sizes_are_pure_and_monotone():
    lib = B.load_library()
    a = lib.cq_rotate_quant_workspace_bytes(16, 4096)
    assert a == lib.cq_rotate_quant_workspace_bytes(16, 4096) and a >= 16 * 4096 * 4
    assert lib.cq_rotate_quant_workspace_bytes(4096, 4096) == 0       # enough tiles: no K split
    assert lib.cq_route_permute_workspace_bytes(2048, 2048, 128, 8) >= (2048 * 8 // 256) * 128 * 4


@pytest.mark.parametrize("name,over", [
    ("tiny", {}), ("mixtral_decode", {}), ("mixtral_decode", dict(group_k=1024)), ("mixtral_decode", dict(index_bits=2)),
    ("mixtral_decode", dict(h_bits=8, r_hadamard=True)), ("dsv2lite", {}), ("qwen3_zipf", {}),
    ("mixtral_decode", dict(H=8192, I=1024, top_k=1)), ("dsv2lite", dict(H=3840, I=2560)),
])
def test_a_workspace_serves_every_smaller_batch(name, over):
    """The queries never fall as the batch grows, whichever kernels the batches take: a workspace sized once, for the
    largest batch, is accepted for all others (a call refuses less than the query of its own batch).  The sizes fell at
    81, 128 and 192 tokens of these shapes, where a batch takes other kernels than a slightly smaller one."""
    c = synth.small_variant(synth.CONFIGS[name], **over)
    lib, G = B.load_library(), c.E + c.S
    weights = [B.CodebookWeights(256, 256, 256, G, n, k, c.group_k, c.index_bits) for n, k in ((2 * c.I, c.H), (c.H, c.I))]
    for split in (None, 256):   # without and with a split copy of the rotation
        L = B.Layer(c.H, c.I, c.E, c.top_k, c.S, c.act_bits, 256, 256, None, *weights, split, c.h_bits, int(c.r_hadamard))
        sizes = [lib.cq_moe_workspace_bytes(ctypes.byref(L), T) for T in range(1, 700)]
        assert sizes[0] > 0 and sizes == sorted(sizes)
        assert lib.cq_moe_forward(ctypes.byref(L), 256, 77, 256, 256, sizes[76] - 1, None) == 4   # CQ_ERR_WORKSPACE
    for W in weights:
        sizes = [lib.cq_grouped_gemm_workspace_bytes(ctypes.byref(W), M) for M in range(1, 700)]
        assert sizes == sorted(sizes)
    sizes = [lib.cq_route_permute_workspace_bytes(T, c.H, c.E, c.top_k) for T in range(1, 2100)]
    assert sizes == sorted(sizes)


@pytest.mark.parametrize("G,N,K,rows,passes", [
    # a product of K = 256 may have 320 units of 64 weight rows: (groups + rows / 32) x N / 64
    (4, 2048, 256, 100, True), (8, 2048, 256, 66, True), (8, 2048, 256, 128, False), (8, 4096, 256, 66, False), (4, 1024, 128, 66, False), (16, 16384, 256, 66, False),
    (8, 4096, 512, 66, False), (8, 2048, 512, 66, True), (32, 1024, 512, 132, True), (32, 1024, 512, 256, False), (64, 2048, 512, 198, False),
    (8, 4096, 1024, 128, True), (128, 2048, 768, 264, False), (16, 1536, 1024, 200, True), (17, 2048, 1024, 480, False),
    (66, 2816, 1408, 512, True), (128, 4096, 1408, 512, True), (66, 2048, 1408, 512, False), (80, 2048, 1408, 480, False),
    (82, 2048, 1408, 480, True), (8, 2048, 1408, 200, True), (128, 1536, 2048, 1024, True), (8, 2048, 2048, 224, False),
])
def test_short_k_streams_in_passes_where_its_units_are_few(G, N, K, rows, passes):
    """Batches of 33 and more tokens with K <= 2048: the product streams in passes (and the layer keeps no second copy of
    its codes) only where few units follow each other on a workgroup, otherwise it is on tiles."""
    lib = B.load_library()
    k = next(k for k in (8, 6, 5, 4, 3, 2, 1) if rows % k == 0 and rows // k > 32)
    T = rows // k
    gu = B.CodebookWeights(256, 256, 256, G, N, K)
    dn = B.CodebookWeights(256, 256, 256, G, K, N // 2)
    L = B.Layer(K, N // 2, G, k, 0, 8, 256, 256, None, gu, dn)
    lay = B.MoeLayout()
    assert lib.cq_moe_workspace_layout(ctypes.byref(L), T, ctypes.byref(lay)) == 0
    assert lay.scale - lay.Q16 == (0 if passes else -(-T * K * 2 // 256) * 256)


def test_prepack_layout_documented_in_header_matches_numpy_model():
    """The tile order and nibble grouping stated in cq.h keep every weight exactly once."""
    rng = np.random.default_rng(5)
    N, K = 64, 128
    idx = rng.integers(0, 256, size=(N, K // 2), dtype=np.uint8)
    packed = Hp.prepack_model(idx)
    # read every weight back through the documented position
    for n in (0, 17, 40, 63):
        for k in (0, 1, 5, 12, 63, 64, 77, 127):
            rb, s, l = n // 32, k // 64, (n % 32) + 32 * ((k % 64) // 32)
            within = k % 32                                   # weight inside the lane's 16-byte piece
            dword, w = within // 8, within % 8
            byte = packed[(rb * (K // 64) + s) * 1024 + l * 16 + dword * 4 + w % 4]
            got = (int(byte) >> (4 * (w // 4))) & 15
            want = (int(idx[n, k // 2]) >> (4 * (k % 2))) & 15
            assert got == want
    assert sorted(np.concatenate([packed & 15, packed >> 4]).tolist()) == \
        sorted(np.concatenate([idx.reshape(-1) & 15, idx.reshape(-1) >> 4]).tolist())


def test_exchanges_within_a_wavefront_are_fenced():
    """Lanes that hand values to each other through LDS without a workgroup barrier use the helper that orders memory: the
    wavefront barrier alone lets the compiler move a load in front of another lane's store."""
    import os
    from paper_2604_10496_amd import build
    for name in sorted(os.listdir(build.CSRC)):
        with open(os.path.join(build.CSRC, name)) as f:
            bare = f.read().count("__builtin_amdgcn_wave_barrier()")
        assert bare == (1 if name == "cq_internal.h" else 0), name


def test_closing_waits_name_the_registers_that_loads_still_target():
    """The last loads of a pipeline from inline assembly are not used by anybody.  Their registers must be operands of what
    waits for them: to the compiler they are free otherwise, and what it keeps in them a late load overwrites."""
    import os
    import re
    from paper_2604_10496_amd import build
    loads = 0
    for name in sorted(os.listdir(build.CSRC)):
        with open(os.path.join(build.CSRC, name)) as f:
            text = f.read()
        calls = name != "cq_async.h" and "load_global_async_s<" in text
        loads += calls
        if not calls and name != "cq_async.h":
            continue
        assert not re.search(r's_waitcnt vmcnt\(0\)"\s*::', text), f"{name}: a closing wait without registers"
        if calls:   # (one closing wait per kernel body that has a ring)
            assert re.search(r's_waitcnt vmcnt\(0\)"\s*:\s*"\+v"', text), f"{name}: no closing wait"
    assert loads >= 2


@pytest.mark.parametrize("G,M,N,K,half", [
    (1, 2048, 4096, 4096, True), (1, 2049, 4096, 4096, False), (1, 384, 28672, 4096, False), (1, 383, 28672, 4096, True),
    (2, 2755, 4096, 4096, False), (8, 5112, 2048, 7168, False), (8, 3904, 2048, 7168, True), (8, 3905, 2048, 7168, False),
    (16, 6144, 1024, 2560, True), (8, 5112, 2048, 2048, True), (8, 3071, 28672, 4096, True), (8, 8192, 28672, 4096, False)])
def test_rule_between_whole_and_half_tiles(G, M, N, K, half):
    """Half tiles for a short K, for fewer than 384 rows per group, and for launches whose half tiles all run at once: one
    that gives some of the 256 compute units two of them is faster on whole tiles, of which they have one each."""
    lib = B.load_library()
    rule = lib._Z23cq_gemm_uses_half_tilesPK19cq_codebook_weightsil
    rule.restype, rule.argtypes = ctypes.c_bool, [ctypes.c_void_p, ctypes.c_int, ctypes.c_long]
    W = B.CodebookWeights(256, 256, None, G, N, K)
    assert rule(ctypes.byref(W), M, M) is half


@pytest.mark.parametrize("T,H,parts,narrow", [
    (128, 8192, 4, True), (129, 8192, 4, False), (384, 8192, 2, False), (512, 7168, 2, False), (128, 6144, 4, True),
    (256, 6144, 4, False), (270, 6144, 2, True), (384, 5120, 2, True), (385, 5120, 2, False), (512, 4096, 2, True),
    (960, 4096, 1, True), (961, 4096, 2, False), (2048, 2048, 1, True), (64, 4096, 16, True), (1025, 4096, 1, False)])
def test_rule_for_the_rotation_in_narrow_tiles(T, H, parts, narrow):
    """Tiles of 64 tokens in half as many parts of K read R twice as often: not where R is wide and the batch has several."""
    lib = B.load_library()
    rule = lib._Z21cq_rotate_split_partsiimPb
    rule.restype, rule.argtypes = ctypes.c_int, [ctypes.c_int, ctypes.c_int, ctypes.c_size_t, ctypes.POINTER(ctypes.c_bool)]
    got = ctypes.c_bool()
    assert (rule(T, H, 1 << 32, ctypes.byref(got)), got.value) == (parts, narrow)


def test_build_reads_spill_counts_from_the_compiler_remarks():
    """build.py refuses kernels with asynchronous register loads that spill; its reader of hipcc's resource
    remarks is checked on a sample of that output."""
    from paper_2604_10496_amd import build
    tag = "[-Rpass-analysis=kernel-resource-usage]"
    sample = [
        f"a.hip:12:1: remark: Function Name: kern_a {tag}",
        "   12 | __global__ void kern_a() {",
        "      | ^",
        f"a.hip:12:1: remark:     VGPRs: 34 {tag}",
        f"a.hip:12:1: remark:     ScratchSize [bytes/lane]: 0 {tag}",
        f"a.hip:12:1: remark:     VGPRs Spill: 0 {tag}",
        "a.hip:40:3: warning: something else",
        f"a.hip:50:1: remark: Function Name: kern_b {tag}",
        "   50 | __global__ void kern_b() {",
        "      | ^",
        f"a.hip:50:1: remark:     ScratchSize [bytes/lane]: 8 {tag}",
        f"a.hip:50:1: remark:     VGPRs Spill: 2 {tag}",
    ]
    usage, rest = build._split_resource_remarks(sample)
    assert usage == {"kern_a": {"VGPRs": 34, "ScratchSize [bytes/lane]": 0, "VGPRs Spill": 0},
                     "kern_b": {"ScratchSize [bytes/lane]": 8, "VGPRs Spill": 2}}
    assert rest == ["a.hip:40:3: warning: something else"]
