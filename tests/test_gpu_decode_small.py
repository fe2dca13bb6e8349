"""Small decode batches: one workgroup per split, merged by the last of each (session, KV head) to
finish, without a second launch.  Against the oracle at the edges of blocks, splits and rows, with
arbitrary workspace contents."""
import ctypes
import math
import os
import re

import numpy as np
import pytest
import torch

from paper_2606_22983_amd import workloads as W
from tests.gpu_util import DevicePool, assert_attn_close, bf16_dev, i32_dev
from tests.test_gpu_decode import _synthetic

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def kv():
    from paper_2606_22983_amd import kv as kv_mod
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    return kv_mod


def _small(kv, dp, q, tables, lens, append, host, ws=None):
    """Tokens per split of the single-launch kernel for this call (ws: its workspace), 0: it takes decode_kernel."""
    n = kv.decode_workspace_bytes(dp.pool, q.shape[0], q.shape[1], tables.shape[1])
    arr = np.ascontiguousarray(lens, dtype=np.int32)
    t = kv.raw_library().ls_internal_small_decode(
        dp.pool.handle, q.shape[0], q.shape[1], tables.shape[1], arr.ctypes.data_as(ctypes.c_void_p) if host else None,
        int(append), ctypes.c_void_p(0 if ws is None else ws.data_ptr()),
        ctypes.c_size_t(n if ws is None else ws.numel() * ws.element_size()), None)
    assert t >= 0
    return t


def _call(kv, dp, q, kn, vn, tables, lens, host, ws, d, lens_host=None):
    out = torch.full(q.shape, float("nan"), dtype=torch.bfloat16, device="cuda")
    lh = None if not host else lens if lens_host is None else lens_host
    kv.paged_attn_decode(dp.pool, 0, bf16_dev(q), i32_dev(tables), i32_dev(lens), 1 / math.sqrt(d), out, ws,
                         None if kn is None else bf16_dev(kn), None if vn is None else bf16_dev(vn),
                         context_lens_host=lh)
    return out


def _tag(name):
    """A constant of the kernel's source."""
    src = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2606_22983_amd", "csrc")
    return int(re.search(r"\b%s = (0x[0-9A-F]+)u" % name, open(os.path.join(src, "decode.hip")).read()).group(1), 16)


def _arrived(n, below=0):
    """An arrival word of count n (n = 0, below > 0: a word that `below` arrivals turn into one), as int64."""
    low, high = _tag("kArrivedLow") + n - below, _tag("kArrivedHigh") + (0xFFFF - n) + below
    return (high << 32 | low) - (1 << 64)


def _workspace(kv, dp, q, tables, fill):
    n = kv.decode_workspace_bytes(dp.pool, q.shape[0], q.shape[1], tables.shape[1])
    ws = torch.empty((n + 7) // 8, dtype=torch.int64, device="cuda")
    ws.fill_(fill)
    return ws


def _unaligned(kv, dp, q, tables):
    n = kv.decode_workspace_bytes(dp.pool, q.shape[0], q.shape[1], tables.shape[1])
    return torch.zeros(n // 8 + 2, dtype=torch.int64, device="cuda")[1:]


CASES = [
    (32, 4, 128, [1789]), (32, 4, 128, [1, 16, 17, 255, 256, 257, 511, 512]), (16, 2, 128, [513, 3000, 1, 767, 768, 769]),
    (8, 1, 128, [16384, 5]), (4, 4, 128, [300, 900, 1023]), (16, 4, 64, [100, 511, 512, 513, 3000]), (8, 8, 64, [1025, 31]),
    (4, 2, 64, [1, 2000]), (8, 1, 64, [8191, 8192, 8193]), (16, 2, 128, list(range(1, 131))),
    # no session is split: any number of workgroups
    (32, 4, 128, list(range(1, 301))), (8, 8, 64, list(range(120, 240))), (8, 2, 128, [1024, 1023, 513] * 60),
]


@pytest.mark.parametrize("host", [False, True])
@pytest.mark.parametrize("append", [False, True])
@pytest.mark.parametrize("hq,hkv,d,lens", CASES)
def test_small_decode_matches_oracle(kv, oracle_lib, hq, hkv, d, lens, append, host):
    rng = np.random.default_rng(sum(lens) + hq)
    lens = np.array(lens, np.int64) - (1 if append else 0)
    pool, tables, q, kn, vn = _synthetic(rng, lens, hq, hkv, d, append)
    dp = DevicePool(kv, pool, d)
    assert _small(kv, dp, q, tables, lens, append, host)
    ref, ref_pool = oracle_lib.decode(pool, 16, d, 0, q, tables, lens, 1 / math.sqrt(d), k_new=kn, v_new=vn,
                                      pool_out=True)
    # Arbitrary contents of the counts: zeros, ones, words that arrivals carry into a count, counts past
    # any call's splits, what the call leaves.
    ws = _workspace(kv, dp, q, tables, 0)
    first = None
    for fill in (0, -1, 0x3F8000003F800000, _arrived(0, 1), _arrived(0, 2), _arrived(0, 3), _arrived(300),
                 _arrived(0xFFFF), None, None):
        if fill is not None:
            ws.fill_(fill)
        out = _call(kv, dp, q, kn, vn, tables, lens, host, ws, d)
        if first is None:
            first = out
            assert_attn_close(out, ref, "small decode %s append=%s host=%s" % (list(lens[:8]), append, host))
        assert torch.equal(out.view(torch.int16), first.view(torch.int16)), fill
    if append:
        assert np.array_equal(dp.host(), ref_pool)
    # A workspace that is only 8-byte aligned takes the other schedule, unless no session is split.
    other_ws = _unaligned(kv, dp, q, tables)
    other = _call(kv, dp, q, kn, vn, tables, lens, host, other_ws, d)
    assert (_small(kv, dp, q, tables, lens, append, host, other_ws) == 0) == (lens.max() + append > _small(
        kv, dp, q, tables, lens, append, host))
    assert_attn_close(other, ref, "8-byte aligned workspace")
    assert kv.ls_device_errors() == 0


@pytest.mark.parametrize("host", [False, True])
def test_small_decode_after_part_of_a_count_was_overwritten(kv, oracle_lib, host):
    """The memory of a finished call's workspace goes to other use, of which stores of one, two or four
    bytes reach the counts, and comes back as a workspace."""
    rng = np.random.default_rng(13)
    lens = np.array([513, 3000, 1, 767, 1600])
    pool, tables, q, _, _ = _synthetic(rng, lens, 16, 2, 128, False)
    dp = DevicePool(kv, pool, 128)
    assert _small(kv, dp, q, tables, lens, False, host)
    ref = oracle_lib.decode(pool, 16, 128, 0, q, tables, lens, 1 / math.sqrt(128))
    ws = _workspace(kv, dp, q, tables, 0)
    first = _call(kv, dp, q, None, None, tables, lens, host, ws, 128)
    assert_attn_close(first, ref, "small decode")
    for dtype, size in ((torch.uint8, 1), (torch.int16, 2), (torch.int32, 4)):
        for at in range(0, 8, size):
            for value in (0, 1, 2, 255 if size == 1 else -1):
                ws.view(dtype)[at // size::128 // size] = value
                ws.view(torch.uint8)[len(lens) * 2 * 128:] = 0xFF                 # no partials of an earlier call
                out = _call(kv, dp, q, None, None, tables, lens, host, ws, 128)
                assert torch.equal(out.view(torch.int16), first.view(torch.int16)), (size, at, value)
    assert kv.ls_device_errors() == 0


def test_small_decode_shapes_share_a_workspace(kv, oracle_lib):
    """Calls of different shapes in turn on one workspace: each finds the others' partials and
    counts where its own counts are."""
    rng = np.random.default_rng(3)
    made = []
    for hq, hkv, d, lens in CASES[:6]:
        lens = np.array(lens, np.int64)
        pool, tables, q, _, _ = _synthetic(rng, lens, hq, hkv, d, False)
        dp = DevicePool(kv, pool, d)
        made.append((dp, q, tables, lens, d, oracle_lib.decode(pool, 16, d, 0, q, tables, lens, 1 / math.sqrt(d))))
    ws = torch.zeros(max(kv.decode_workspace_bytes(m[0].pool, len(m[3]), m[1].shape[1], m[2].shape[1]) for m in made),
                     dtype=torch.uint8, device="cuda")
    for rep in range(3):
        for i, (dp, q, tables, lens, d, ref) in enumerate(made):
            out = _call(kv, dp, q, None, None, tables, lens, bool((rep + i) & 1), ws, d)
            assert_attn_close(out, ref, "shared workspace, call %d.%d" % (rep, i))
    assert kv.ls_device_errors() == 0


def test_small_decode_errors_and_other_device_lengths(kv, oracle_lib):
    rng = np.random.default_rng(4)
    lens = np.array([700, 1500, 40, 600])
    pool, tables, q, _, _ = _synthetic(rng, lens, 16, 2, 128, False)
    dp = DevicePool(kv, pool, 128)
    ws = _workspace(kv, dp, q, tables, 0)
    kv.ls_device_errors()
    # an empty context: zeros, flagged; the others as usual
    dev = lens.copy()
    dev[2] = 0
    out = _call(kv, dp, q, None, None, tables, dev, False, ws, 128)
    assert bool((out[2] == 0).all()) and kv.ls_device_errors() == kv.LS_DEVERR_LENGTH
    keep = [0, 1, 3]
    ref = oracle_lib.decode(pool, 16, 128, 0, q, tables, lens, 1 / math.sqrt(128))
    assert_attn_close(out[keep], ref[keep], "beside an empty context")
    # device lengths shorter than the host's rows
    short = np.array([300, 1, 40, 513])
    out = _call(kv, dp, q, None, None, tables, short, True, ws, 128, lens_host=lens)
    assert_attn_close(out, oracle_lib.decode(pool, 16, 128, 0, q, tables, short, 1 / math.sqrt(128)), "shorter")
    assert kv.ls_device_errors() == 0
    # longer than the host's rows: flagged
    _call(kv, dp, q, None, None, tables, lens, True, ws, 128, lens_host=np.array([700, 100, 40, 600]))
    assert kv.ls_device_errors() == kv.LS_DEVERR_LENGTH
    _call(kv, dp, q, None, None, tables, lens, True, ws, 128, lens_host=np.array([200, 100, 40, 250]))
    assert kv.ls_device_errors() == kv.LS_DEVERR_LENGTH
    # and the next call counts as usual
    out = _call(kv, dp, q, None, None, tables, lens, True, ws, 128)
    assert_attn_close(out, ref, "after a flagged call")
    # a block id outside the pool: flagged, its keys absent
    bad = tables.copy()
    bad[1, 3] = 1 << 29
    _call(kv, dp, q, None, None, bad, lens, False, ws, 128)
    assert kv.ls_device_errors() == kv.LS_DEVERR_BLOCK_ID


@pytest.mark.parametrize("kernel", ["small", "persistent"])
@pytest.mark.parametrize("host", [False, True])
@pytest.mark.parametrize("hq,hkv,d", [(16, 2, 128), (8, 4, 64)])
def test_bad_block_ids_and_empty_contexts_in_either_kernel(kv, oracle_lib, hq, hkv, d, host, kernel):
    """Ids outside the pool, at a split's first block and inside one, and a context without a key, in the
    single-launch kernel and in decode_kernel: flagged, the block's keys absent, the row zero."""
    rng = np.random.default_rng(hq + d)
    lens = np.array([700, 1500, 40, 3000, 1200])
    pool, tables, q, _, _ = _synthetic(rng, lens, hq, hkv, d, False)
    dp = DevicePool(kv, pool, d)
    ws = _workspace(kv, dp, q, tables, -1) if kernel == "small" else _unaligned(kv, dp, q, tables)
    assert bool(_small(kv, dp, q, tables, lens, False, host, ws)) == (kernel == "small")
    bad, gone, left = tables.copy(), np.full_like(tables, -1), lens.copy()
    bad[1, 3], bad[3, 0], bad[3, 100] = 1 << 29, -7, pool.shape[1]
    for s in range(5):
        keep = [j for j in range(tables.shape[1]) if not (bad[s, j] != tables[s, j])]
        gone[s, :len(keep)] = tables[s, keep]
        left[s] -= 16 * (tables.shape[1] - len(keep))
    ref = oracle_lib.decode(pool, 16, d, 0, q, gone, left, 1 / math.sqrt(d))
    kv.ls_device_errors()
    out = _call(kv, dp, q, None, None, bad, lens, host, ws, d)
    assert kv.ls_device_errors() == kv.LS_DEVERR_BLOCK_ID
    assert_attn_close(out, ref, "beside absent blocks")
    # device lengths with an empty context (host lengths say otherwise, or nothing)
    dev = lens.copy()
    dev[2] = 0
    out = _call(kv, dp, q, None, None, tables, dev, host, ws, d, lens_host=lens)
    assert kv.ls_device_errors() == kv.LS_DEVERR_LENGTH and bool((out[2] == 0).all())
    keep = [0, 1, 3, 4]
    ref = oracle_lib.decode(pool, 16, d, 0, q, tables, lens, 1 / math.sqrt(d))
    assert_attn_close(out[keep], ref[keep], "beside an empty context")


@pytest.mark.parametrize("kernel", ["small", "persistent"])
def test_scores_at_infinity_and_nan_in_either_kernel(kv, oracle_lib, kernel):
    """Splits whose scores are all -inf for half of the heads (8 * -3e38 is past the fp32 range) leave the
    result to the others; a NaN key, or one at +inf, makes its heads NaN and no others."""
    rng = np.random.default_rng(31)
    lens, hq, hkv, d = np.array([3000, 600]), 16, 2, 128
    pool, tables, q, _, _ = _synthetic(rng, lens, hq, hkv, d, False)
    q[:, :, 0] = 0
    q[:, ::2, 0] = W.to_bf16(np.float32(8.0))
    t = np.arange(200, 2000)
    pool[0, tables[0, t // 16], 0, :, (t % 16) * 8] = W.to_bf16(np.float32(-3e38))
    dp = DevicePool(kv, pool, d)
    ws = _workspace(kv, dp, q, tables, -1) if kernel == "small" else _unaligned(kv, dp, q, tables)
    assert bool(_small(kv, dp, q, tables, lens, False, True, ws)) == (kernel == "small")
    ref = oracle_lib.decode(pool, 16, d, 0, q, tables, lens, 1 / math.sqrt(d))
    assert_attn_close(_call(kv, dp, q, None, None, tables, lens, True, ws, d), ref, "scores at -inf")
    for bits, key in ((0x7FC0, 2900), (0x7F80, 100)):
        p2 = pool.copy()
        p2[0, tables[0, key // 16], 0, 1, (key % 16) * 8 + 1] = bits          # dim 1 of KV head 1's key
        q2 = q.copy()
        q2[:, :, 1] = W.to_bf16(np.float32(1.0))
        ref2 = oracle_lib.decode(pool, 16, d, 0, q2, tables, lens, 1 / math.sqrt(d))
        dp2 = DevicePool(kv, p2, d)
        out = _call(kv, dp2, q2, None, None, tables, lens, True, ws, d)
        assert bool(out[0, 8:].isnan().all())
        assert_attn_close(out[0, :8], ref2[0, :8], "beside a key of %#x" % bits)
        assert_attn_close(out[1], ref2[1], "another session")
    assert kv.ls_device_errors() == 0
