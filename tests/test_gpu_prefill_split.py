"""Prefill calls whose query tiles are too few to fill the GPU: their keys are split over
workgroups and merged (host lengths and a full-size workspace).  Against the oracle, where parts
end at tile edges, inside the causal diagonal or hold no key of a row."""
import math

import numpy as np
import pytest
import torch

from paper_2606_22983_amd import workloads as W
from tests.gpu_util import DevicePool, assert_attn_close, bf16_dev, i32_dev, scale_keys
from tests.test_gpu_prefill import _case

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def kv():
    from paper_2606_22983_amd import kv as kv_mod
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    return kv_mod


def _call(kv, dp, q, kn, vn, n, c, tables, d, ws_bytes, lens_dev=None):
    n_dev, c_dev = (n, c) if lens_dev is None else lens_dev
    cu = np.concatenate([[0], np.cumsum(n_dev)]).astype(np.int32)
    out = torch.full(q.shape, float("nan"), dtype=torch.bfloat16, device="cuda")
    ws = torch.full((ws_bytes,), 0xFF, dtype=torch.uint8, device="cuda")       # NaN partials, garbage counters
    kv.paged_attn_prefill(dp.pool, 0, bf16_dev(q), i32_dev(cu), i32_dev(c_dev), int(np.max(n)), i32_dev(tables),
                          1 / math.sqrt(d), out, None if kn is None else bf16_dev(kn),
                          None if vn is None else bf16_dev(vn), lens_host=np.stack([n, c], 1), workspace=ws)
    # The pieces' region (256 rows of maximum and sum) is written exactly when something was split.
    split = not bool((ws[kv.PREFILL_COUNTER_BYTES:] == 0xFF).all())
    return out, cu, split


# (hq, hkv, d, n, c): one short turn over a long context (many parts); a first turn whose parts end
# inside the causal diagonal; one new token; lengths one past a key tile; several uneven turns with
# an empty one; one query head per KV head; a second wave of which only a remainder is split.
@pytest.mark.parametrize("hq,hkv,d,n,c", [
    (32, 4, 128, [301], [9043]), (4, 1, 128, [2048], [0]), (8, 1, 128, [1], [16384]), (8, 2, 64, [65], [4097]),
    (16, 2, 128, [33, 0, 257, 8], [5000, 7000, 3001, 12]), (8, 8, 64, [700], [2000]),
    (4, 4, 128, [256, 255], [2047, 3000]),
    (32, 4, 128, [560, 560, 560, 560], [6300, 6100, 6049, 5500])])
def test_split_prefill_matches_oracle(kv, oracle_lib, hq, hkv, d, n, c):
    rng = np.random.default_rng(hq * 7 + n[0])
    n, c = np.array(n), np.array(c)
    pool, tables, q, kn, vn = _case(rng, n, c, hq, hkv, d)
    dp = DevicePool(kv, pool, d)
    out, cu, split = _call(kv, dp, q, kn, vn, n, c, tables, d, kv.PREFILL_WORKSPACE_BYTES)
    ref, ref_pool = oracle_lib.prefill(pool, 16, d, 0, q, kn, vn, cu, c, tables, 1 / math.sqrt(d), pool_out=True)
    assert split
    assert_attn_close(out, ref, "split prefill n=%s c=%s" % (n, c))
    assert np.array_equal(dp.host(), ref_pool)
    # Without an append (the K/V is in the pool now) the counters are cleared by their own kernel.
    again, _, _ = _call(kv, dp, q, None, None, n, c, tables, d, kv.PREFILL_WORKSPACE_BYTES)
    assert torch.equal(out.view(torch.int16), again.view(torch.int16))
    # A counters-only workspace is still taken, and splits nothing.
    whole, _, split = _call(kv, dp, q, None, None, n, c, tables, d, kv.PREFILL_COUNTER_BYTES)
    assert not split
    assert_attn_close(whole, ref, "unsplit prefill n=%s c=%s" % (n, c))
    assert kv.ls_device_errors() == 0


# Turns that end around the edges of a wave's 32 rows, a query tile and a key tile, where waves have
# no rows or stop before the workgroup's last key tile (G = 1 and 8); and the same with one long turn,
# where padding is a small share and every wave keeps to the workgroup's tiles.
@pytest.mark.parametrize("mode", ["device", "host", "workspace"])
@pytest.mark.parametrize("hq,hkv,d,n,c", [
    (8, 8, 64, [31, 32, 33, 255, 256, 257, 1], [0, 0, 31, 0, 64, 63, 0]),
    (4, 4, 128, [31, 33, 63, 65, 129, 255, 257, 300], [0, 1, 0, 64, 0, 15, 0, 100]),
    (16, 2, 128, [3, 4, 5, 31, 33, 9], [0, 61, 64, 100, 0, 127]),
    (2, 2, 64, [1700, 30], [0, 40])])
def test_prefill_waves_without_rows_or_keys(kv, oracle_lib, hq, hkv, d, n, c, mode):
    rng = np.random.default_rng(hkv + n[0])
    n, c = np.array(n), np.array(c)
    pool, tables, q, kn, vn = _case(rng, n, c, hq, hkv, d)
    dp = DevicePool(kv, pool, d)
    cu = np.concatenate([[0], np.cumsum(n)]).astype(np.int32)
    out = torch.full(q.shape, float("nan"), dtype=torch.bfloat16, device="cuda")
    ws = torch.full((kv.PREFILL_WORKSPACE_BYTES,), 0x5A, dtype=torch.uint8, device="cuda")
    ws = ws if mode == "workspace" else None
    kv.paged_attn_prefill(dp.pool, 0, bf16_dev(q), i32_dev(cu), i32_dev(c), int(n.max()), i32_dev(tables),
                          1 / math.sqrt(d), out, bf16_dev(kn), bf16_dev(vn),
                          lens_host=None if mode == "device" else np.stack([n, c], 1), workspace=ws)
    ref = oracle_lib.prefill(pool, 16, d, 0, q, kn, vn, cu, c, tables, 1 / math.sqrt(d))
    assert_attn_close(out, ref, "turns %s over %s" % (n, c))
    assert kv.ls_device_errors() == 0


# Keys whose scores overflow to -inf for the rows with q[0] = 8, and are ordinary for those with q[0] = 0
# (8 * -3e38 is past the fp32 range): the first 32 keys of every key tile but the first, so that every
# part after the first begins with them; a run of key tiles that holds whole parts; everything but the
# first key tile and the turn itself.
@pytest.mark.parametrize("where", ["unit", "parts", "rest"])
@pytest.mark.parametrize("hq,hkv,d,n,c", [(16, 2, 128, [40], [6000]), (8, 2, 64, [65, 3], [4097, 2500]),
                                          (4, 4, 128, [300], [3000])])
def test_split_prefill_of_scores_that_overflow(kv, oracle_lib, hq, hkv, d, n, c, where):
    rng = np.random.default_rng(11)
    n, c = np.array(n), np.array(c)
    pool, tables, q, kn, vn = _case(rng, n, c, hq, hkv, d)
    for s in range(len(n)):
        t = np.arange(int(c[s]))
        t = t[{"unit": (t >= 64) & (t % 64 < 32), "parts": (t >= 640) & (t < 640 + 64 * ((c[s] - 700) // 64)),
               "rest": t >= 64}[where]]
        pool[0, tables[s, t // 16], 0, :, (t % 16) * 8] = W.to_bf16(np.float32(-3e38))      # dim 0 of the K rows
    q[:, :, 0] = 0
    q[::2, :, 0] = W.to_bf16(np.float32(8.0))
    dp = DevicePool(kv, pool, d)
    out, cu, split = _call(kv, dp, q, kn, vn, n, c, tables, d, kv.PREFILL_WORKSPACE_BYTES)
    ref = oracle_lib.prefill(pool, 16, d, 0, q, kn, vn, cu, c, tables, 1 / math.sqrt(d))
    assert split
    assert_attn_close(out, ref, "%s of scores at -inf" % where)
    whole, _, split = _call(kv, dp, q, None, None, n, c, tables, d, kv.PREFILL_COUNTER_BYTES)
    assert not split
    assert_attn_close(whole, ref, "%s of scores at -inf, unsplit" % where)
    assert kv.ls_device_errors() == 0


@pytest.mark.parametrize("bits", [0x7FC0, 0x7F80])
def test_split_prefill_of_nan_and_inf_keys(kv, oracle_lib, bits):
    """A NaN key, or one whose score is +inf, late in the context: the rows that are NaN unsplit are
    NaN, the others as without it."""
    rng = np.random.default_rng(12)
    n, c, d = np.array([40]), np.array([6000]), 128
    pool, tables, q, kn, vn = _case(rng, n, c, 16, 2, d)
    q[:, :, 0] = W.to_bf16(np.float32(1.0))
    ref = oracle_lib.prefill(pool, 16, d, 0, q, kn, vn, np.array([0, 40]), c, tables, 1 / math.sqrt(d))
    pool[0, tables[0, 4000 // 16], 0, 1, (4000 % 16) * 8] = bits                 # KV head 1 alone
    dp = DevicePool(kv, pool, d)
    out, _, split = _call(kv, dp, q, kn, vn, n, c, tables, d, kv.PREFILL_WORKSPACE_BYTES)
    whole, _, _ = _call(kv, dp, q, None, None, n, c, tables, d, kv.PREFILL_COUNTER_BYTES)
    assert split and torch.equal(out.isnan(), whole.isnan()) and bool(out[:, 8:].isnan().all())
    assert_attn_close(out[:, :8], ref[:, :8], "beside a key of %#x" % bits)


@pytest.mark.parametrize("shape", ["rising", "spike", "falling"])
def test_split_prefill_of_peaky_scores(kv, oracle_lib, shape):
    """Parts whose maxima differ by orders of magnitude."""
    rng = np.random.default_rng(5)
    n, c, d = np.array([40]), np.array([6000]), 128
    pool, tables, q, kn, vn = _case(rng, n, c, 16, 2, d)
    scale_keys(pool, tables, c, shape)
    dp = DevicePool(kv, pool, d)
    out, cu, split = _call(kv, dp, q, kn, vn, n, c, tables, d, kv.PREFILL_WORKSPACE_BYTES)
    assert split
    assert_attn_close(out, oracle_lib.prefill(pool, 16, d, 0, q, kn, vn, cu, c, tables, 1 / math.sqrt(d)), shape)


def test_split_prefill_with_other_device_lengths(kv, oracle_lib):
    """The plan is the host's, the lengths are the device's: a shorter device turn and context (all
    its tiles, and parts, shrink) give the device lengths' result."""
    rng = np.random.default_rng(6)
    n, c, d = np.array([200]), np.array([5000]), 128
    pool, tables, q, kn, vn = _case(rng, n, c, 16, 2, d)
    dp = DevicePool(kv, pool, d)
    dn, dc = np.array([70]), np.array([100])
    out, cu, split = _call(kv, dp, q, kn, vn, n, c, tables, d, kv.PREFILL_WORKSPACE_BYTES, lens_dev=(dn, dc))
    assert split
    ref = oracle_lib.prefill(pool, 16, d, 0, q[:70], kn[:70], vn[:70], cu, dc, tables, 1 / math.sqrt(d))
    assert_attn_close(out[:70], ref, "shorter device lengths")
    assert bool(torch.isnan(out[70:]).all())                  # rows past the turn are not written
    kv.ls_device_errors()


def test_split_prefill_with_a_negative_device_context(kv, oracle_lib):
    """A device context below zero leaves every part of that session without key tiles: the call
    ends, flags it, and the other session's rows are as usual."""
    rng = np.random.default_rng(9)
    n, c, d = np.array([200, 90]), np.array([5000, 4000]), 128
    pool, tables, q, kn, vn = _case(rng, n, c, 16, 2, d)
    ref = oracle_lib.prefill(pool, 16, d, 0, q, kn, vn, np.array([0, 200, 290]), c, tables, 1 / math.sqrt(d))
    kv.ls_device_errors()
    for c0 in (-1, -150, -300, -(1 << 30)):
        dp = DevicePool(kv, pool, d)
        out, _, split = _call(kv, dp, q, kn, vn, n, c, tables, d, kv.PREFILL_WORKSPACE_BYTES,
                              lens_dev=(n, np.array([c0, 4000])))
        assert split and kv.ls_device_errors() & kv.LS_DEVERR_LENGTH
        assert_attn_close(out[200:], ref[200:], "beside a context of %d" % c0)


def test_split_prefill_with_device_contexts_past_the_table(kv):
    """A device context longer than the table: flagged, and the blocks past the table are absent
    (keys and values of zero) in whichever part they fall, as they are unsplit."""
    rng = np.random.default_rng(10)
    n, c, d = np.array([40, 60]), np.array([2000, 1900]), 128
    pool, tables, q, kn, vn = _case(rng, n, c, 16, 2, d)
    pool[(pool & 0x7FFF) > 0x7F80] = 0                        # (no NaN past the host's contexts)
    dp = DevicePool(kv, pool, d)
    for c0 in (2500, 8000, 20000):
        dev = (n, np.array([c0, 1900]))
        kv.ls_device_errors()
        out, _, split = _call(kv, dp, q, kn, vn, n, c, tables, d, kv.PREFILL_WORKSPACE_BYTES, lens_dev=dev)
        assert split and kv.ls_device_errors() & kv.LS_DEVERR_LENGTH
        whole, _, split = _call(kv, dp, q, kn, vn, n, c, tables, d, kv.PREFILL_COUNTER_BYTES, lens_dev=dev)
        assert not split and kv.ls_device_errors() & kv.LS_DEVERR_LENGTH
        assert_attn_close(out, whole.float().cpu().numpy(), "context of %d in a table of %d" % (c0, 16 * tables.shape[1]))


def test_split_prefill_replays_from_a_graph(kv):
    rng = np.random.default_rng(8)
    n, c, d, hq, hkv = np.array([100]), np.array([8000]), 128, 32, 4
    pool, tables, q, kn, vn = _case(rng, n, c, hq, hkv, d)
    dp = DevicePool(kv, pool, d)
    eager, cu, split = _call(kv, dp, q, kn, vn, n, c, tables, d, kv.PREFILL_WORKSPACE_BYTES)
    assert split
    ws = torch.empty(kv.PREFILL_WORKSPACE_BYTES, dtype=torch.uint8, device="cuda")
    args = [bf16_dev(q), i32_dev(cu), i32_dev(c), 100, i32_dev(tables), 1 / math.sqrt(d), torch.empty_like(eager),
            bf16_dev(kn), bf16_dev(vn)]
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        kv.paged_attn_prefill(dp.pool, 0, *args, lens_host=np.stack([n, c], 1), workspace=ws)
    for rep in range(3):
        ws.fill_(0x77)
        args[6].fill_(0)
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(args[6].view(torch.int16), eager.view(torch.int16)), rep
