"""Host-only checks of the C ABI: the library loads, exports every function that
include/hack.h declares, and rejects bad arguments before launching anything.
No call here reaches the GPU."""
import ctypes
import os
import re

import pytest

from oracle import hack_oracle as O

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HEADER = os.path.join(ROOT, "include", "hack.h")

hk = pytest.importorskip("paper_2502_03589_amd.hack")


@pytest.fixture(scope="module")
def lib():
    if not os.path.exists(hk.library_path()):
        pytest.skip("libhack.so not built (run __graft_entry__.build())")
    return hk.lib()


def declared_functions():
    text = open(HEADER).read()
    text = re.sub(r"/\*.*?\*/", "", text, flags=re.S)
    return sorted(set(re.findall(r"\b(hack_[a-z0-9_]+)\s*\(", text)))


def test_every_declared_symbol_is_exported(lib):
    names = declared_functions()
    assert len(names) >= 10
    for n in names:
        assert hasattr(lib, n), n
    assert set(names) == set(hk.EXPORTS)


def test_layout_make_validation(lib):
    good = hk.hack_kv_layout_make(128, 8, 2, 32, 256)
    assert good.sum_bytes == 1 and good.qp_bits == 8
    assert hk.hack_kv_layout_make(128, 8, 2, 128, 256).sum_bytes == 2     # 9-bit sums -> 2 bytes
    assert hk.hack_kv_layout_make(128, 8, 4, 64, 256).sum_bytes == 2
    bad = [
        (128, 8, 3, 32, 256), (128, 8, 8, 32, 256), (128, 8, 2, 48, 256), (100, 8, 2, 32, 256),
        (128, 0, 2, 32, 256), (128, 8, 2, 32, 100), (128, 8, 2, 32, 0), (512, 8, 2, 32, 256),
    ]
    for args in bad:
        with pytest.raises(hk.HackError) as e:
            hk.hack_kv_layout_make(*args)
        assert e.value.status == 1
    for qp in (0, 2, 5, 7, 16):
        with pytest.raises(hk.HackError):
            hk.hack_kv_layout_make(128, 8, 2, 32, 256, qp_bits=qp)
    assert hk.hack_kv_layout_make(128, 8, 2, 32, 256, qp_bits=4).qp_bits == 4
    with pytest.raises(hk.HackError):
        hk.hack_kv_layout_make(128, 8, 2, 32, 256, rounding=7)
    assert lib.hack_kv_layout_make(None, 128, 8, 2, 32, 256, 8, 0, 0) == 1


@pytest.mark.parametrize("bits,pi", [(2, 32), (4, 32), (2, 64), (4, 64), (2, 128), (2, 16)])
def test_section_sizes_closed_form(lib, bits, pi):
    d, H, pt, pages = 128, 8, 256, 5
    lay = hk.hack_kv_layout_make(d, H, bits, pi, pt)
    P = d // pi
    sb = O.sum_bytes(bits, pi)
    expect = {
        hk.K_CODES: pages * H * pt * d * bits // 8,
        hk.K_META: pages * H * pt * P * 4,
        hk.K_SUMS: pages * H * pt * P * sb,
        hk.V_CODES: pages * H * (pt // pi) * d * pi * bits // 8,
        hk.V_META: pages * H * (pt // pi) * d * 4,
        hk.V_SUMS: pages * H * (pt // pi) * d * sb,
    }
    for sec, n in expect.items():
        assert hk.hack_kv_bytes(lay, pages, sec) == n
    assert hk.hack_kv_bytes(lay, 3, hk.V_TAIL) == 3 * H * pi * d * 2
    assert hk.hack_kv_bytes(lay, -1, hk.K_CODES) == -1
    assert hk.hack_kv_bytes(lay, 1, 99) == -1
    # bytes per token per kv head (K + V, excluding the fp16 open block): b=2, pi=32 -> 104
    per_tok = sum(hk.hack_kv_bytes(lay, 1, s) for s in range(6)) / (H * pt)
    assert per_tok == (d * bits // 8 + P * (4 + sb)) + d * (pi * bits // 8 + 4 + sb) / pi


def test_compression_ratio_of_format(lib):
    """Sec. 7.2: codes + fp16 min/scale at 2 bits and Pi = 64 are ~15% of fp16 KV."""
    lay = hk.hack_kv_layout_make(128, 1, 2, 64, 64)
    codes_meta = sum(hk.hack_kv_bytes(lay, 1, s) for s in (hk.K_CODES, hk.K_META, hk.V_CODES, hk.V_META))
    fp16 = 2 * 64 * 128 * 2
    assert codes_meta / fp16 == 0.15625


class _Fake:
    """A cache struct whose pointers are non-null but never dereferenced."""
    def __init__(self, pages=4, table=None, mbps=0):
        c = hk.hack_kv_cache()
        for i, n in enumerate(hk.SECTIONS):
            setattr(c, n, 0x1000 * (i + 1))
        c.num_pages = pages
        if table:
            c.block_table_dev = 0x9000
            c.max_blocks_per_seq = mbps
        self.struct = c


def test_argument_errors_before_launch(lib):
    lay = hk.hack_kv_layout_make(128, 2, 2, 32, 128)
    L = ctypes.byref(lay)
    fake = _Fake(pages=4)
    C = ctypes.byref(fake.struct)
    p = ctypes.c_void_p(0x5000)
    # null inputs
    assert lib.hack_quantize(L, C, None, p, p, 2, 10, None) == 1
    # capacity: contiguous capacity is page_tokens = 128
    assert lib.hack_quantize(L, C, p, p, p, 2, 129, None) == 3
    assert lib.hack_append(L, C, p, p, p, 2, 128, 0, None) == 3
    assert lib.hack_append(L, C, p, p, p, 2, 10, 5, None) == 1      # bad tail mode
    # contiguous cache needs one page per sequence
    assert lib.hack_quantize(L, C, p, p, p, 5, 10, None) == 1
    # paged capacity = pages per sequence * page_tokens
    paged = _Fake(pages=4, table=True, mbps=3)
    assert lib.hack_quantize(L, ctypes.byref(paged.struct), p, p, p, 2, 3 * 128 + 1, None) == 3
    # decode: workspace too small, unsupported shapes
    ws = hk.hack_decode_workspace_bytes(lay, 2, 8, 100)
    assert ws > 0
    assert lib.hack_attend_decode(L, C, p, 8, p, 2, 100, 0, p, p, ws - 1, None) == 4
    assert lib.hack_attend_decode(L, C, p, 8, p, 2, 100, 0, p, None, ws, None) == 4
    assert lib.hack_attend_decode(L, C, p, 7, p, 2, 100, 0, p, p, ws, None) == 1      # H_q % H_kv
    assert lib.hack_attend_decode(L, C, p, 2 * 16, p, 2, 100, 0, p, p, 10 ** 9, None) == 2   # group 16
    lay64 = hk.hack_kv_layout_make(64, 2, 2, 32, 128)
    assert lib.hack_attend_decode(ctypes.byref(lay64), C, p, 8, p, 2, 100, 0, p, p, 10 ** 9, None) == 2
    lay128 = hk.hack_kv_layout_make(128, 2, 2, 128, 128)
    assert lib.hack_attend_prefill(ctypes.byref(lay128), C, p, 8, 2, 129, 1, p, None) == 3  # validated
    assert lib.hack_attend_prefill(L, C, p, 8, 2, 129, 1, p, None) == 3
    # a sequence per grid row/plane: batch is bounded by the grid's y/z extent
    assert lib.hack_attend_decode(L, C, p, 8, p, 65536, 100, 0, p, p, 10 ** 12, None) == 2
    assert lib.hack_attend_prefill(L, C, p, 8, 65536, 100, 1, p, None) == 2
    # decode step: capacity counts the appended token, length arrays must differ,
    # workspace is sized for max_len + 1, paged caches need pages of 4 * partition
    p2 = ctypes.c_void_p(0x6000)
    wss = hk.hack_decode_workspace_bytes(lay, 2, 8, 101)
    assert lib.hack_decode_step(L, C, p, p, p, 8, p, p2, 2, 128, 0, p, p, 10 ** 9, None) == 3
    assert lib.hack_decode_step(L, C, p, p, p, 8, p, p, 2, 100, 0, p, p, 10 ** 9, None) == 1
    assert lib.hack_decode_step(L, C, None, p, p, 8, p, p2, 2, 100, 0, p, p, 10 ** 9, None) == 1
    assert lib.hack_decode_step(L, C, p, p, p, 8, p, p2, 2, 100, 7, p, p, 10 ** 9, None) == 1
    assert lib.hack_decode_step(L, C, p, p, p, 8, p, p2, 2, 100, 0, p, p, wss - 1, None) == 4
    lay_pg = hk.hack_kv_layout_make(128, 2, 2, 32, 64)
    paged64 = _Fake(pages=4, table=True, mbps=3)
    assert lib.hack_attend_decode(ctypes.byref(lay_pg), ctypes.byref(paged64.struct), p, 8, p, 2, 100, 0, p, p,
                                  10 ** 9, None) == 2
    # zero-sized work is a no-op that succeeds without launching
    assert lib.hack_decode_step(L, C, p, p, p, 8, p, p2, 0, 10, 0, p, p, 10 ** 9, None) == 0
    assert lib.hack_quantize(L, C, p, p, p, 0, 10, None) == 0
    assert lib.hack_attend_prefill(L, C, p, 8, 2, 0, 1, p, None) == 0


def test_quantize_grid_limit_checked_before_launch(lib):
    """At partitions >= 64 every V block is one workgroup: a cache with more than
    2^31 - 1 blocks is rejected before anything is launched."""
    lay = hk.hack_kv_layout_make(128, 8, 2, 64, 1 << 16)
    big = _Fake(pages=1 << 18)
    p = ctypes.c_void_p(0x5000)
    assert lib.hack_quantize(ctypes.byref(lay), ctypes.byref(big.struct), p, p, p, 1 << 18, 1 << 16, None) == 2


def test_workspace_grows_with_context(lib):
    lay = hk.hack_kv_layout_make(128, 8, 2, 32, 256)
    a = hk.hack_decode_workspace_bytes(lay, 16, 32, 4096)
    b = hk.hack_decode_workspace_bytes(lay, 16, 32, 131072)
    assert 0 < a <= b
    assert hk.hack_decode_workspace_bytes(lay, 16, 31, 4096) == -1
    # chunk records: at most 65535 chunks per sequence (the grid's z extent),
    # each holding max, sum and O per query head
    big = hk.hack_decode_workspace_bytes(lay, 1, 32, 2 ** 31 - 1)
    assert 0 < big <= 8 * 65535 * 4 * (4 + 128) * 4 + 4096


def _planned_splits(ws, pairs, group, head_groups, head_dim=128):
    """Chunks per sequence of a decode plan, read back from its workspace size
    (counters first, 256-byte aligned, then one record of max, sum and O per chunk
    and query head)."""
    counters = (pairs * head_groups * 4 + 255) // 256 * 256
    per_split = pairs * group * (4 + head_dim) * 4
    records = ws - counters
    assert records % per_split == 0
    return records // per_split


@pytest.mark.parametrize("bits,batch,hq,max_len,splits", [
    (2, 64, 64, 32769, 6),    # ragged 70B-shaped batch: even share 343 spans -> chunks of 48 spans
    (4, 4, 32, 131136, 17),   # long context at 4 bits: share 65 spans -> chunks of 64 (one round)
    (2, 4, 32, 131136, 24),   # long context at 2 bits: share 43 spans kept
])
def test_decode_chunk_plan(lib, bits, batch, hq, max_len, splits):
    """Split-K chunking of decode: an even share of the resident workgroup slots at
    max_len, at most 64 spans of 4 partitions (128 tokens at partition 32), and 48 spans
    when the share exceeds 128 spans (a batch of many long sequences)."""
    lay = hk.hack_kv_layout_make(128, 8, bits, 32, 256)
    ws = hk.hack_decode_workspace_bytes(lay, batch, hq, max_len)
    pairs, group = batch * 8, hq // 8
    assert _planned_splits(ws, pairs, group, (group + 3) // 4) == splits


@pytest.mark.parametrize("bits,pi,batch,hq,hkv,max_len,splits", [
    (2, 32, 1, 1, 1, 256, 1),     # two spans: one chunk, nothing to merge
    (2, 32, 16, 16, 2, 512, 1),   # four spans, one a wave
    (4, 64, 1, 32, 8, 1280, 3),   # five spans of 8 groups: chunks of two
    (2, 32, 4, 32, 8, 1000, 4),   # eight spans of 32 groups
    (2, 32, 16, 16, 2, 1024, 2),  # eight spans of 64 groups: one span a wave again
    (2, 32, 1, 32, 8, 4096, 8),   # 32 spans: one span a wave
    (2, 64, 7, 64, 8, 3001, 4),   # even share of three spans: 448 workgroups of three, not 336 of four
    (2, 32, 32, 32, 8, 4096, 3),  # even share of eleven spans: kept
])
def test_decode_short_chunk_plan(lib, bits, pi, batch, hq, hkv, max_len, splits):
    """Chunks of short sequences: a span per wave (four), fewer only for five to eight spans of
    few groups and where an even share of three spans fills the chip better."""
    lay = hk.hack_kv_layout_make(128, hkv, bits, pi, 4 * pi)
    pairs, group = batch * hkv, hq // hkv
    up = lambda n: -(-n // 256) * 256
    ws = hk.hack_decode_workspace_bytes(lay, batch, hq, max_len)
    assert ws == up(pairs * ((group + 3) // 4) * 4) + up(pairs * splits * group * (4 + 128) * 4)


def test_status_strings(lib):
    for st in range(6):
        assert len(hk.hack_status_string(st)) > 0
    assert hk.hack_status_string(99) == "unknown status"


@pytest.mark.parametrize("bits,pi", [(2, 32), (4, 64), (2, 128)])
def test_summation_elimination_off_layout(lib, bits, pi):
    """Sums not cached (Sec. 5.3's summation elimination switched off): the sum sections
    have no bytes, every other section is unchanged, and it can be switched back."""
    d, H, pt, pages = 128, 8, 256, 3
    on = hk.hack_kv_layout_make(d, H, bits, pi, pt)
    off = hk.hack_kv_layout_make(d, H, bits, pi, pt, sums_cached=False)
    assert off.sum_bytes == 0 and on.sum_bytes == O.sum_bytes(bits, pi)
    for sec in range(7):
        want = 0 if sec in (hk.K_SUMS, hk.V_SUMS) else hk.hack_kv_bytes(on, pages, sec)
        assert hk.hack_kv_bytes(off, pages, sec) == want
    hk.hack_kv_layout_set_sums(off, True)
    assert off.sum_bytes == on.sum_bytes
    assert lib.hack_kv_layout_set_sums(ctypes.byref(off), 2) == 1
    assert lib.hack_kv_layout_set_sums(None, 0) == 1


def test_summation_elimination_off_arguments(lib):
    """Without cached sums the sum pointers may be null; prefill and the debug exports
    (which read the cached sums) report UNSUPPORTED before any launch."""
    lay = hk.hack_kv_layout_make(128, 2, 2, 32, 128, sums_cached=False)
    L = ctypes.byref(lay)
    fake = _Fake(pages=4)
    fake.struct.k_sums = None
    fake.struct.v_sums = None
    C = ctypes.byref(fake.struct)
    p = ctypes.c_void_p(0x5000)
    assert lib.hack_attend_prefill(L, C, p, 8, 2, 100, 1, p, None) == 2
    assert lib.hack_debug_qk_products(L, C, p, 8, p, 2, 100, p, p, p, None) == 2
    assert lib.hack_debug_pv_products(L, C, p, p, 8, p, 2, 100, p, p, None) == 2
    assert lib.hack_quantize(L, C, p, p, p, 2, 129, None) == 3  # validated (capacity), not rejected
    on = hk.hack_kv_layout_make(128, 2, 2, 32, 128)
    assert lib.hack_quantize(ctypes.byref(on), C, p, p, p, 2, 10, None) == 1  # cached sums need pointers


def test_partition128_workspace_follows_its_plan(lib):
    """Partition 128 chunks sequences into whole 512-token spans (one 128-token block
    per wave) so that the grid holds 4 (2-bit) or 2 (4-bit) workgroups per compute
    unit of 256: at decode_llama8b_l4096's shapes that is 8 (2-bit) or 4 (4-bit)
    chunks per sequence; one int32 counter per (sequence, kv head, group of four query
    heads) comes first, 256-byte aligned, then records of 4 + 128 floats per (sequence,
    kv head, chunk, query head)."""
    def expect(B, H, G, L, per_cu):
        span, pairs, nhg = 512, B * H, (G + 3) // 4
        spans_seq = -(-L // span)
        wg = min(max(-(-(spans_seq * pairs * nhg) // (256 * per_cu)), 1), 64)
        splits = -(-L // (wg * span))
        rec = -(-(pairs * splits * G * (4 + 128) * 4) // 256) * 256
        return -(-(pairs * nhg * 4) // 256) * 256 + rec, splits
    for bits, per_cu in ((2, 4), (4, 2)):
        lay = hk.hack_kv_layout_make(128, 8, bits, 128, 4096)
        ws, splits = expect(16, 8, 4, 4096, per_cu)
        assert splits == (8 if bits == 2 else 4)
        assert hk.hack_decode_workspace_bytes(lay, 16, 32, 4096) == ws
        for B, H, G, L in ((1, 1, 1, 1), (3, 2, 8, 5000), (1, 8, 6, 131072), (64, 8, 4, 300)):
            lay = hk.hack_kv_layout_make(128, H, bits, 128, 512)
            assert hk.hack_decode_workspace_bytes(lay, B, H * G, L) == expect(B, H, G, L, per_cu)[0]


def test_noalloc_limits_checked_before_launch(lib):
    """hack_attend_decode_noalloc takes its split-K state from a static scratch of 65536
    counters and 16 MiB of chunk records: larger shapes get HACK_ERR_WORKSPACE on the
    host, other argument errors the same statuses as hack_attend_decode, and a batch of
    0 succeeds, all before anything touches the device."""
    lay = hk.hack_kv_layout_make(128, 8, 2, 32, 256)
    L = ctypes.byref(lay)
    paged = _Fake(pages=4, table=True, mbps=512)  # capacity 131072 tokens per sequence
    C = ctypes.byref(paged.struct)
    p = ctypes.c_void_p(0x5000)
    # 8192 sequences x 8 kv heads x 2 four-head groups = 131072 counters
    assert lib.hack_attend_decode_noalloc(L, C, p, 64, p, 8192, 1024, 0, p, None) == 4
    # 64 sequences of 131072 tokens, group 8: chunk records beyond 16 MiB
    full = hk.hack_decode_workspace_bytes(lay, 64, 64, 131072)
    assert full - 256 * ((64 * 8 * 2 * 4 + 255) // 256) > 16 << 20
    assert lib.hack_attend_decode_noalloc(L, C, p, 64, p, 64, 131072, 0, p, None) == 4
    assert lib.hack_attend_decode_noalloc(L, C, p, 7, p, 2, 100, 0, p, None) == 1       # H_q % H_kv
    assert lib.hack_attend_decode_noalloc(L, C, p, 16, p, 2, 100, 5, p, None) == 1      # tail mode
    assert lib.hack_attend_decode_noalloc(L, C, p, 16, p, 2, 100, 0, None, None) == 1   # no output
    assert lib.hack_attend_decode_noalloc(L, C, p, 16, p, 2, 131073, 0, p, None) == 3   # capacity
    assert lib.hack_attend_decode_noalloc(L, C, p, 16, p, 0, 100, 0, p, None) == 0
