"""Host-side checks of the C-ABI library that need no GPU: it loads, exports
every symbol the header declares, and rejects bad arguments before touching the
device."""
import inspect
import os
import re
import shutil
import subprocess
import sys

import numpy as np
import pytest

from paper_2404_12457_amd import binding as B

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def lib():
    from paper_2404_12457_amd import build

    if not (os.path.exists(B.LIB_PATH) and os.path.exists(build.CALLS)):
        build.build()
    return B.load()


@pytest.mark.parametrize("header_name,exports", [("ragc.h", "binding"), ("ragc_ctl.h", "ctl")])
def test_every_declared_symbol_is_exported(lib, header_name, exports):
    from paper_2404_12457_amd import ctl

    header = open(os.path.join(ROOT, "include", header_name)).read()
    header = re.sub(r"/\*.*?\*/", "", header, flags=re.S)
    names = set(re.findall(r"\b(ragc_[a-z_0-9]+)\s*\(", header))
    assert names == set(B.EXPORTS if exports == "binding" else ctl.EXPORTS)
    for n in names:
        assert getattr(lib, n) is not None


def test_version_and_kv_bytes_per_token_match_the_model_table(lib):
    assert B.ragc_version() >= 100
    for line in open(os.path.join(ROOT, "tests", "golden", "kv_bytes_per_token.txt")):
        if line.startswith("#") or not line.strip():
            continue
        name, layers, hq, hkv, mib = line.split()
        assert B.ragc_kv_bytes_per_token(int(layers), int(hkv), 128, B.RAGC_DTYPE_BF16) == float(mib) * 2**20, name
    assert B.ragc_kv_bytes_per_token(0, 8, 128, 1) == 0 and B.ragc_kv_bytes_per_token(32, 8, 128, 7) == 0


A = 0x10000  # a fake, aligned, non-NULL address: validation never dereferences device pointers


def _pool(**kw):
    args = dict(k=A, v=A, num_blocks=64, kv_heads=2, head_dim=128, dtype=B.RAGC_DTYPE_BF16)
    args.update(kw)
    return B.make_pool(**args)


def _batch(p=(10,), n=(5,), stride=4, table=None, dev=A):
    hp, hn = np.asarray(p, np.int32), np.asarray(n, np.int32)
    hs = np.concatenate([[0], np.cumsum(np.maximum(hn, 0))]).astype(np.int32)
    b = B.make_batch(len(p), stride, dev, dev, dev, dev, hp, hn, hs, table)
    return b, (hp, hn, hs, table)


def _attn_code(pool, batch, q=A, k=A, v=A, o=A, hq=8, scale=0.1, flags=0):
    with pytest.raises(B.RagcError) as e:
        B.ragc_prefill_attn(pool, batch, q, k, v, o, hq, scale, flags)
    return e.value.code


def test_attention_argument_errors(lib):
    b, keep = _batch()
    assert _attn_code(_pool(k=None), b) == B.RAGC_ERR_NULL
    assert _attn_code(_pool(block_size=32), b) == B.RAGC_ERR_SHAPE
    assert _attn_code(_pool(head_dim=96), b) == B.RAGC_ERR_SHAPE
    assert _attn_code(_pool(dtype=3), b) == B.RAGC_ERR_SHAPE
    assert _attn_code(_pool(block_stride_elems=100), b) == B.RAGC_ERR_SHAPE
    assert _attn_code(_pool(k=A + 2), b) == B.RAGC_ERR_ALIGN
    assert _attn_code(_pool(), b, hq=3) == B.RAGC_ERR_SHAPE
    assert _attn_code(_pool(), b, scale=0.0) == B.RAGC_ERR_SHAPE
    assert _attn_code(_pool(), b, scale=float("nan")) == B.RAGC_ERR_SHAPE
    assert _attn_code(_pool(), b, flags=0x80) == B.RAGC_ERR_SHAPE
    assert _attn_code(_pool(), b, q=None) == B.RAGC_ERR_NULL
    assert _attn_code(_pool(), b, o=A + 4) == B.RAGC_ERR_ALIGN
    b2, keep2 = _batch(dev=None)
    assert _attn_code(_pool(), b2) == B.RAGC_ERR_NULL
    b3, keep3 = _batch(p=(60,), n=(10,), stride=4)  # 70 tokens need 5 entries
    assert _attn_code(_pool(), b3) == B.RAGC_ERR_RANGE
    b4, keep4 = _batch(p=(-1,))
    assert _attn_code(_pool(), b4) == B.RAGC_ERR_RANGE
    tbl = np.array([[1, 64, 0, 0]], np.int32)  # block 64 does not exist
    b5, keep5 = _batch(p=(20,), n=(5,), table=tbl)
    assert _attn_code(_pool(), b5) == B.RAGC_ERR_RANGE
    assert "block_table[1] = 64" in B.ragc_last_error()
    hp = np.asarray([1], np.int32)
    b6 = B.make_batch(1, 4, None, None, None, None, None, hp, hp, None)  # no host copy and no device array to read it from
    with pytest.raises(B.RagcError) as e:
        B.ragc_prefill_attn_workspace(_pool(), b6, 8)
    assert e.value.code == B.RAGC_ERR_NULL and "prefix_len" in B.ragc_last_error()
    with pytest.raises(B.RagcError) as e:  # the entry point that may not read anything back wants all three host copies
        B.ragc_prefill_attn_static(_pool(), B.make_batch(1, 4, A, A, A, A, None, hp, hp, None), A, A, A, A, 8, 0.1)
    assert e.value.code == B.RAGC_ERR_NULL
    with pytest.raises(B.RagcError) as e:
        B.ragc_prefill_attn_static(_pool(), b, A, A, A, A, 8, 0.1, B.RAGC_ATTN_VALIDATE)
    assert e.value.code == B.RAGC_ERR_SHAPE


def test_append_wants_rows_packed_in_request_order(lib):
    """The append kernel finds a row's request by searching new_start, so the offsets must be the
    running sum of new_len; attention takes any offsets.  Both checks happen before any launch."""
    hp, hn = np.asarray([10, 20, 5], np.int32), np.asarray([5, 0, 7], np.int32)
    for hs, ok in ((np.asarray([0, 5, 5, 12], np.int32), True), (np.asarray([3, 8, 8, 15], np.int32), True),
                   (np.asarray([0, 6, 6, 13], np.int32), False), (np.asarray([7, 0, 0, 0], np.int32), False)):
        b = B.make_batch(3, 4, A, A, A, A, hp, hn, hs, None)
        if ok:
            continue  # would launch: covered by the GPU tests
        with pytest.raises(B.RagcError) as e:
            B.ragc_kv_append(_pool(), b, A, A)
        assert e.value.code == B.RAGC_ERR_RANGE and "packed in request order" in B.ragc_last_error()


def test_debug_plan_override_changes_the_workspace_and_rejects_bad_values(lib):
    one, keep = _batch(p=(4096,), n=(16,), stride=300)
    pool = _pool(num_blocks=512)
    auto = B.ragc_prefill_attn_workspace(pool, one, 8)
    try:
        B.ragc_debug_set_attn_plan(-1, 3)  # two 32-row items, two kv heads, three copies
        assert B.ragc_debug_get_attn_plan(pool, one, 8) == (32, 8, 3)
        assert B.ragc_prefill_attn_workspace(pool, one, 8) == 3 * 2 * 2 * 32 * (128 + 2) * 4
        B.ragc_debug_set_attn_plan(0, 3)  # one 128-row item
        assert B.ragc_debug_get_attn_plan(pool, one, 8) == (128, 4, 3)
        assert B.ragc_prefill_attn_workspace(pool, one, 8) == 3 * 2 * 128 * (128 + 2) * 4
        B.ragc_debug_set_attn_plan(0, 1)
        assert B.ragc_debug_get_attn_plan(pool, one, 8) == (128, 4, 1)
        assert B.ragc_prefill_attn_workspace(pool, one, 8) == 0
        for bad in ((2, 0), (-2, 0), (0, 17), (0, -1)):
            with pytest.raises(B.RagcError) as e:
                B.ragc_debug_set_attn_plan(*bad)
            assert e.value.code == B.RAGC_ERR_SHAPE
        assert B.ragc_prefill_attn_workspace(pool, one, 8) == 0  # a rejected call leaves the setting alone
    finally:
        B.ragc_debug_set_attn_plan(-1, 0)
    assert B.ragc_prefill_attn_workspace(pool, one, 8) == auto


def _plan(p, n, hq, hkv, d=128, flags=0, dtype=B.RAGC_DTYPE_BF16):
    """(rows per work item, waves, copies) of the library's own choice, 256 CUs when no GPU is visible (an MI355X has as
    many); the workspace is one partial result per work item, copy and kv head, and nothing where there is one copy."""
    b, keep = _batch(p=p, n=n, stride=1200)
    pool = _pool(num_blocks=4096, kv_heads=hkv, head_dim=d, dtype=dtype)
    rows, waves, copies = B.ragc_debug_get_attn_plan(pool, b, hq, flags)
    items = sum(-(-(x * (hq // hkv)) // rows) for x in n) if rows else 0
    want = items * copies * hkv * rows * (d + 2) * 4 if copies > 1 else 0
    assert B.ragc_prefill_attn_workspace(pool, b, hq, flags) == want
    # never more than one 128-row partial result per CU
    assert want <= 256 * 128 * (d + 2) * 4
    return rows, waves, copies


def test_key_split_rule(lib):
    """Copies of a 32-row item: at least two key tiles for each of eight waves, one workgroup per CU, at most 16; one up to
    1408 keys."""
    assert _plan((4096,) * 4, (1,) * 4, 64, 8) == (32, 8, 8)       # 32 workgroups, 129 tiles: every CU gets one
    assert _plan((1024,), (100,), 32, 32) == (32, 8, 1)            # 128 workgroups, 36 tiles
    assert _plan((1308,), (100,), 32, 32) == (32, 8, 1)            # 44 tiles
    assert _plan((1309,), (100,), 32, 32) == (32, 8, 2)            # 45 tiles
    assert _plan((2048,) * 2, (1,) * 2, 32, 8) == (32, 8, 4)       # 16 workgroups, 65 tiles
    assert _plan((16384,), (1,), 32, 8) == (32, 8, 16)             # capped
    assert _plan((16384,), (1,), 32, 8, flags=B.RAGC_ATTN_NO_SPLIT) == (32, 8, 1)
    assert _plan((1024,) * 8, (1,) * 8, 32, 32) == (32, 8, 1)      # 256 workgroups already
    assert _plan((100,), (20,), 8, 8) == (32, 8, 1)                # four tiles: nothing to split
    assert _plan((10, 0), (0, 0), 8, 8) == (0, 0, 0)


@pytest.mark.parametrize("p,n,hq,hkv,d,want", [
    # 32 rows per request: always the 32-row kernel; one more row and a full chip of 128-row items: the 128-row kernel
    ((300,) * 256, (8,) * 256, 8, 2, 128, (32, 4, 1)),
    ((300,) * 256, (9,) * 256, 8, 2, 128, (128, 4, 1)),
    # fewer 128-row items than CUs: the 32-row kernel up to two of its workgroups per CU
    ((300,), (1024,), 32, 8, 128, (128, 8, 1)),                      # 256 items of 128 rows
    ((300,), (960,), 16, 8, 128, (32, 4, 1)),                        # 120 and 480
    ((300,), (1056,), 16, 8, 128, (128, 8, 1)),                      # 136 and 528
    # one to two 128-row items per CU, half empty: the 32-row kernel, up to three and short keys: shared CUs, above: one each
    ((300,) * 9, (64,) * 9, 32, 32, 128, (128, 4, 1)),               # 288 and 576
    ((300,) * 10, (40,) * 10, 32, 32, 64, (128, 8, 1)),              # 320 and 640 at head_dim 64, all of one length
    ((50,) * 16, (17,) * 16, 32, 16, 128, (128, 8, 1)),              # 256 and 512: exactly one item per CU
    ((50,) * 17, (9,) + (8,) * 16, 64, 16, 128, (32, 4, 1)),         # 272 and 288
    ((50,) * 17, (9,) * 17, 64, 16, 128, (128, 4, 1)),               # 272 and 544
    ((50,) * 17, (9,) * 17, 60, 15, 128, (32, 4, 1)),                # 255 and 510
    ((960,) * 9, (64,) * 9, 32, 32, 128, (128, 4, 1)),               # 1024 keys
    ((961,) * 9, (64,) * 9, 32, 32, 128, (128, 8, 1)),               # 1025 keys
    # ragged batches of head_dim 64
    ((1900, 300, 16, 700, 15, 0), (130, 60, 100, 90, 64, 130), 32, 8, 64, (32, 4, 1)),
    # a little over one 32-row workgroup per CU, thousands of keys, one length: split or whole 128-row items
    ((4445,) * 3, (46,) * 3, 64, 8, 128, (128, 4, 3)),               # 72 and 288
    ((2000,) * 3, (46,) * 3, 64, 8, 128, (32, 4, 1)),                # 2046 keys: four waves instead
    ((4445, 3000, 3000), (46,) * 3, 64, 8, 128, (32, 4, 1)),         # not of one length, mean 0.78 of the longest
    ((4445, 2000, 2000), (46,) * 3, 64, 8, 128, (32, 8, 1)),         # less
    ((3200,) * 20, (23,) * 20, 40, 8, 128, (128, 8, 1)),             # 160 and 320: nothing to split
    # row tiles of a request on several XCDs
    ((6833,) * 8, (17,) * 8, 8, 2, 128, (32, 8, 4)),                 # five copies would fit, four share an L2
    ((5666,) * 9, (6,) * 9, 28, 4, 128, (128, 4, 7)),                # two copies leave CUs idle
    ((2081,) * 9, (6,) * 9, 28, 4, 128, (32, 8, 2)),
    ((7876,) * 3, (92,) * 3, 8, 2, 128, (128, 4, 14)),               # three copies fit, 73 MB would be read again
    ((7876,), (92,), 8, 2, 128, (32, 8, 10)),                        # 24 MB
    # decode steps of head_dim 64
    ((4000,) * 66, (1,) * 66, 40, 8, 64, (128, 4, 1)),               # 528 of one length
    ((4000,) * 65 + (2000,) * 9, (1,) * 74, 40, 8, 64, (32, 4, 1)),  # 592, not of one length
    ((4000,) * 81, (1,) * 81, 40, 8, 64, (32, 4, 1)),                # 648
    ((4000,) * 34, (1,) * 34, 40, 8, 64, (32, 4, 1)),                # 272 of one length
    ((4000,) * 20 + (2000,) * 14, (1,) * 34, 40, 8, 64, (32, 8, 1)),
    # decode steps of head_dim 128
    ((2000,) * 64, (1,) * 64, 64, 8, 128, (32, 4, 1)),
    ((2000,) * 30 + (700,) * 34, (1,) * 64, 64, 8, 128, (32, 8, 1)),
    ((1500,) * 10 + (500,) * 54, (1,) * 64, 64, 8, 128, (32, 4, 1)),  # fewer than 1024 keys on average
])
def test_plan_on_both_sides_of_its_lines(lib, p, n, hq, hkv, d, want):
    assert _plan(p, n, hq, hkv, d) == want


def _product(p, n, hq, hkv, d=128, dtype=B.RAGC_DTYPE_BF16):
    b, keep = _batch(p, n, stride=max((x + y + 15) // 16 for x, y in zip(p, n)) or 1)
    return B.ragc_debug_get_attn_product(_pool(num_blocks=1 << 20, kv_heads=hkv, head_dim=d, dtype=dtype), b, hq)


@pytest.mark.parametrize("p,n,hq,hkv,d,want", [
    ((93,) * 96, (32,) * 96, 32, 8, 128, 16),             # 768 items of 128 rows, four 32-row ones each: 1500 keys per CU
    ((92,) * 96, (32,) * 96, 32, 8, 128, 32),             # 1488
    ((0,) * 96, (32,) * 96, 32, 8, 128, 32),              # prompts of one tile
    ((93,) * 95, (32,) * 95, 32, 8, 128, 32),             # 760 items
    ((2744,) * 4, (256,) * 4, 32, 8, 128, 16),            # 256 items, four 32-row ones each: 12000 keys per CU
    ((2743,) * 4, (256,) * 4, 32, 8, 128, 32),            # 11996
    ((5744,) * 4, (256,) * 4, 32, 8, 64, 0),              # head_dim 64
    ((1024,), (100,), 32, 32, 128, 0),                    # 32-row items
    ((4445,) * 3, (46,) * 3, 64, 8, 128, 0),              # split items
    ((10, 0), (0, 0), 8, 8, 128, 0),
])
def test_product_on_both_sides_of_its_lines(lib, p, n, hq, hkv, d, want):
    assert _product(p, n, hq, hkv, d) == want
    assert _product(p, n, hq, hkv, d, dtype=B.RAGC_DTYPE_F32) == 0
    try:
        for rows in (16, 32):
            assert B.ragc_debug_set_attn_product(rows) == 0
            assert _product(p, n, hq, hkv, d) == (rows if want else 0)
        for bad in (-1, 1, 64):
            with pytest.raises(B.RagcError):
                B.ragc_debug_set_attn_product(bad)
        with pytest.raises(B.RagcError):
            _product(p, n, hq + 1, hkv + hkv, d)
    finally:
        B.ragc_debug_set_attn_product(0)


def test_fp32_plan(lib):
    assert _plan((300,), (64,), 32, 8, dtype=B.RAGC_DTYPE_F32) == (16, 8, 1)    # 128 workgroups
    assert _plan((300,), (129,), 32, 8, dtype=B.RAGC_DTYPE_F32) == (16, 4, 1)   # 264


def test_size_limits_and_workspace_errors(lib):
    many, keep = _batch(p=(0,) * 65536, n=(1,) * 65536, stride=1)
    assert _attn_code(_pool(), many) == B.RAGC_ERR_SHAPE  # more requests than a work item can name
    huge, keep2 = _batch(p=(0,), n=(2_000_000,), stride=125_000)
    assert _attn_code(_pool(), huge, hq=16) == B.RAGC_ERR_RANGE  # 16 M rows: more than 65535 row tiles
    assert "too large" in B.ragc_last_error()
    # one request with a long prefix is split along its keys: the workspace is then mandatory, and without a split it is not
    one, keep3 = _batch(p=(4096,), n=(16,), stride=300)
    need = B.ragc_prefill_attn_workspace(_pool(num_blocks=512), one, 8)
    assert need == 8 * 2 * 2 * 32 * (128 + 2) * 4  # eight copies of two 32-row items, two kv heads
    assert B.ragc_prefill_attn_workspace(_pool(num_blocks=512), one, 8, B.RAGC_ATTN_NO_SPLIT) == 0
    assert B.ragc_prefill_attn_workspace(_pool(num_blocks=512, dtype=B.RAGC_DTYPE_F32), one, 8) == 0
    for ws, nbytes, code in ((None, 0, B.RAGC_ERR_WORKSPACE), (A, need - 1, B.RAGC_ERR_WORKSPACE), (A + 16, need, B.RAGC_ERR_ALIGN)):
        with pytest.raises(B.RagcError) as e:
            B.ragc_prefill_attn(_pool(num_blocks=512), one, A, A, A, A, 8, 0.1, 0, ws, nbytes)
        assert e.value.code == code
    with pytest.raises(B.RagcError) as e:
        B.ragc_prefill_attn_workspace(_pool(num_blocks=512), one, 3)
    assert e.value.code == B.RAGC_ERR_SHAPE


def test_empty_work_returns_ok_without_a_device(lib):
    b, keep = _batch(p=(10, 3), n=(0, 0))
    assert B.ragc_prefill_attn(_pool(), b, None, None, None, None, 8, 0.1) == 0
    assert B.ragc_kv_append(_pool(), b, None, None) == 0
    b0 = B.make_batch(0, 0, None, None, None, None, None, None, None, None)
    assert B.ragc_prefill_attn(_pool(), b0, None, None, None, None, 8, 0.1) == 0
    ids = np.zeros(0, np.int32)
    assert B.ragc_kv_swap(_pool(), A, A, 2 * 16 * 128, 4, ids, ids, B.RAGC_SWAP_TO_DEVICE) == 0
    assert B.ragc_kv_gather(_pool(), b, 0, 0, None, None) == 0


def _swap_code(pool, hk=A, hv=A, stride=2 * 16 * 128, slots_n=4, dev=(1,), slots=(0,), direction=0, flags=0):
    with pytest.raises(B.RagcError) as e:
        B.ragc_kv_swap(pool, hk, hv, stride, slots_n, np.asarray(dev, np.int32), np.asarray(slots, np.int32), direction, flags)
    return e.value.code


def test_swap_and_gather_argument_errors(lib):
    assert _swap_code(_pool(), hk=None) == B.RAGC_ERR_NULL
    assert _swap_code(_pool(), stride=100) == B.RAGC_ERR_SHAPE
    assert _swap_code(_pool(), direction=2) == B.RAGC_ERR_SHAPE
    assert _swap_code(_pool(), flags=9) == B.RAGC_ERR_SHAPE
    assert _swap_code(_pool(), dev=(64,)) == B.RAGC_ERR_RANGE
    assert _swap_code(_pool(), slots=(4,)) == B.RAGC_ERR_RANGE
    assert _swap_code(_pool(), dev=(1, 1), slots=(0, 1), direction=0) == B.RAGC_ERR_RANGE  # two writes to block 1
    assert _swap_code(_pool(), dev=(1, 2), slots=(3, 3), direction=1) == B.RAGC_ERR_RANGE  # two writes to slot 3
    assert _swap_code(_pool(), hv=A + 8) == B.RAGC_ERR_ALIGN
    b, keep = _batch()
    with pytest.raises(B.RagcError) as e:
        B.ragc_kv_gather(_pool(), b, 1, 4, A, A)
    assert e.value.code == B.RAGC_ERR_RANGE
    with pytest.raises(B.RagcError) as e:
        B.ragc_kv_gather(_pool(), b, 0, 65, A, A)
    assert e.value.code == B.RAGC_ERR_RANGE


def test_missing_library_fails_loudly(monkeypatch, tmp_path):
    monkeypatch.setattr(B, "_lib", None)
    monkeypatch.setattr(B, "LIB_PATH", str(tmp_path / "nope.so"))
    with pytest.raises(RuntimeError, match="no fallback"):
        B.ragc_version()


@pytest.mark.parametrize("p,n,hq,hkv,d,want", [
    ((300,), (160,), 32, 8, 128, (32, 8, 1)),             # head_dim 128: 320 workgroups of 16 rows
    ((300,), (156,), 32, 8, 128, (16, 4, 1)),             # 312
    ((10,), (160,), 32, 8, 128, (32, 8, 1)),              # 170 keys
    ((100,) * 16, (11,) * 16, 32, 8, 128, (16, 4, 1)),    # 384, and 256 of 32 rows: half empty
    ((0,) * 3, (64,) * 3, 32, 8, 128, (16, 4, 1)),        # 384 of 64 keys, 192 of 32 rows
    ((0,) * 5, (64,) * 5, 32, 8, 128, (32, 4, 1)),        # 640, 320
    ((300,), (132,), 32, 8, 64, (32, 8, 1)),              # head_dim 64: 264
    ((30,), (132,), 32, 8, 64, (16, 4, 1)),               # of 162 keys
    ((300,), (300,), 32, 8, 64, (16, 4, 1)),              # 600
    ((300,), (576,), 32, 8, 64, (32, 4, 1)),              # 1152
])
def test_fp32_plan_on_both_sides_of_its_lines(lib, p, n, hq, hkv, d, want):
    assert _plan(p, n, hq, hkv, d, dtype=B.RAGC_DTYPE_F32) == want


@pytest.mark.parametrize("p,n,d,want", [
    ((300,) * 3, (81,) * 3, 128, (16, 4, 1)),     # 504 workgroups of 16 rows and 264 of 32: one round of two per CU either way
    ((300,) * 3, (85,) * 3, 128, (32, 4, 1)),     # 528 and 264: two rounds against one
    ((300,) * 6, (81,) * 6, 128, (16, 4, 1)),     # 1008 and 528
    ((300,) * 6, (85,) * 6, 128, (32, 4, 1)),     # 1056 and 528: three against two
    ((0,) * 48, (16,) * 48, 64, (32, 4, 1)),      # head_dim 64, few keys: 1536 and 768: two rounds of four per CU against one of three
    ((0,) * 49, (16,) * 49, 64, (16, 4, 1)),      # 1568 and 784
    ((79,) * 49, (16,) * 49, 64, (16, 4, 1)),     # 95 keys
    ((80,) * 49, (16,) * 49, 64, (32, 4, 1)),     # 96
])
def test_fp32_plan_counts_rounds(lib, p, n, d, want):
    assert _plan(p, n, 32, 8, d, dtype=B.RAGC_DTYPE_F32) == want


def _outcome(f, *args, **kwargs):
    try:
        return f(*args, **kwargs)
    except Exception as e:
        return type(e), str(e)


@pytest.mark.parametrize("args,kwargs", [
    (("pool", "empty", A, A, A, A, 8, 0.125), {}),
    (("pool", "empty", A, A, A, A, 8), dict(softmax_scale=0.125, stream=0, flags=1, workspace=None, workspace_bytes=0)),
    (("pool", "batch", A, A, A, A + 1, 8, 0.125), {}),                       # misaligned
    (("pool", "batch", A, A, A, A, 9, 0.125), {}),                           # heads
    (("pool", "batch", None, A, A, A, 8, 0.125), {}),
    ((None, "batch", A, A, A, A, 8, 0.125), {}),
    (("pool", None, A, A, A, A, 8, 0.125), {}),
    (("pool", "batch", A, A, A, A, 8, float("nan")), {}),
    (("pool", "batch", A, A, A, A, 8, 0.125, 1 << 31), {}),                  # unknown flag
    (("pool", "batch", np.zeros(3), A, A, A, np.int64(9), 1), {}),           # an array, a numpy number, a whole scale
    (("batch", "pool", A, A, A, A, 8, 0.125), dict(bad=1)),
    (("pool", "batch", A, A, A, A, 8.0, 0.125), {}),                         # no whole number
    (("pool", "batch", A, A, A, A, 8, "x"), {}),
    (("pool", "batch", "q", A, A, A, 8, 0.125), {}),
    ((b"pool", "batch", A, A, A, A, 8, 0.125), {}),
    (("pool", "batch", A, A, A, A), {}),
    (("pool", "batch", A, A, A, A, 8, 0.125, 0, None, 0, 0, 0), {}),
    (("pool", "batch", A, A, A, A, 8, 0.125), dict(pool=1)),
    (("pool", "batch", A, A, A, A, 1 << 40, 0.125), dict(workspace_bytes=-1)),
])
def test_calls_marshalled_in_c_behave_as_through_ctypes(lib, args, kwargs):
    empty, k0 = _batch(p=(), n=(), stride=1)
    batch, k1 = _batch()
    named = {"pool": _pool(), "empty": empty, "batch": batch}
    args = [named.get(a, a) if isinstance(a, str) else a for a in args]
    assert _outcome(B.ragc_prefill_attn, *args, **kwargs) == _outcome(B._ctypes_calls[0], *args, **kwargs)


def test_append_marshalled_in_c_behaves_as_through_ctypes(lib):
    empty, k0 = _batch(p=(), n=(), stride=1)
    batch, k1 = _batch()
    for args, kwargs in [((_pool(), empty, A, A), {}), ((_pool(), empty, A), dict(v_new=A, stream=0)), ((_pool(), batch, A + 1, A), {}),
                         ((_pool(), batch, None, A), {}), ((None, batch, A, A), {}), ((_pool(), A), {}), ((_pool(), batch, A, A, 1.5), {}),
                         ((_pool(), batch, A, A), dict(flags=1))]:
        assert _outcome(B.ragc_kv_append, *args, **kwargs) == _outcome(B._ctypes_calls[1], *args, **kwargs)


def test_calls_marshalled_in_c_show_their_arguments(lib):
    for f, g in zip((B.ragc_prefill_attn, B.ragc_kv_append), B._ctypes_calls):
        got, want = inspect.signature(f).parameters, inspect.signature(g).parameters
        assert [(p.name, p.default) for p in got.values()] == [(p.name, p.default) for p in want.values()]


AFTER_IMPORT = """
import shutil, sys, warnings
import numpy as np
from paper_2404_12457_amd import binding as B, build
try:
    B.load()
    sys.exit("loaded without a library")
except RuntimeError as e:
    assert "no fallback" in str(e), e
early = B.ragc_kv_append
shutil.copy(sys.argv[1], B.LIB_PATH)
if sys.argv[2] == "built":
    shutil.copy(sys.argv[3], build.CALLS)
elif sys.argv[2] == "broken":
    open(build.CALLS, "wb").write(b"no library")
with warnings.catch_warnings(record=True) as seen:
    warnings.simplefilter("always")
    B.load()
zero = np.zeros(1, np.int32)
batch = B.make_batch(0, 1, 65536, 65536, 65536, 65536, zero, zero, zero)
pool = B.make_pool(65536, 65536, 4, 2, 64, B.RAGC_DTYPE_F32)
assert B.ragc_prefill_attn(pool, batch, 65536, 65536, 65536, 65536, 2, 0.5) == 0
assert B.ragc_kv_append(pool, batch, 65536, 65536) == early(pool, batch, 65536, 65536) == 0
print(type(B.ragc_prefill_attn).__name__, *[str(w.message) for w in seen])
"""


@pytest.mark.parametrize("calls", ["built", "absent", "broken"])
def test_libraries_that_appear_after_the_import(lib, tmp_path, calls):
    """Importing the binding of a tree that is not built yet, building, loading, all in one process; and a tree whose C
    extension is missing or does not load: the calls go through ctypes, and a warning says why."""
    from paper_2404_12457_amd import build

    package = tmp_path / "paper_2404_12457_amd"
    package.mkdir()
    for name in ("__init__.py", "binding.py", "build.py"):
        shutil.copy(os.path.join(os.path.dirname(B.__file__), name), package)
    r = subprocess.run([sys.executable, "-c", AFTER_IMPORT, B.LIB_PATH, calls, build.CALLS], cwd=tmp_path, capture_output=True, text=True,
                       env={k: v for k, v in os.environ.items() if k != "PYTHONPATH"}, timeout=100)
    assert r.returncode == 0, r.stderr
    want = {"built": ("builtin_function_or_method",), "absent": ("function", "_calls"), "broken": ("function", os.path.basename(build.CALLS))}
    assert all(x in r.stdout for x in want[calls]) and ("ctypes" in r.stdout) == (calls != "built"), r.stdout
