"""Kernels on CU-masked streams: the persistent grids are sized to the CUs the
stream may use, and the results do not depend on it."""
import math

import numpy as np
import pytest
import torch

from paper_2606_22983_amd import workloads as W
from tests.gpu_util import (DevicePool, assert_attn_close, bf16_dev, cu_masked_stream, destroy_stream, host_bits,
                            i32_dev, log)
from tests.test_gpu_decode import _synthetic
from tests.test_gpu_prefill import _case

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def kv():
    from paper_2606_22983_amd import kv as kv_mod
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    return kv_mod


def _decode(kv, dp, case, q, tables, lens, stream, ws=None):
    s, hq, d = q.shape
    out = torch.empty((s, hq, d), dtype=torch.bfloat16, device="cuda")
    if ws is None:
        ws = torch.zeros(kv.decode_workspace_bytes(dp.pool, s, hq, tables.shape[1]),
                         dtype=torch.uint8, device="cuda")
    kv.paged_attn_decode(dp.pool, 0, q, tables, lens, case.scale, out, ws, stream=stream)
    return out, ws


def test_the_current_stream_is_torchs(kv, monkeypatch):
    """Both ways to the current stream's handle, on the default stream and on another."""
    other = torch.cuda.Stream()
    for way in ("private", "public"):
        if way == "public":
            monkeypatch.setattr(kv, "_raw_stream", None)
        assert kv._stream(None) == torch.cuda.current_stream().cuda_stream
        with torch.cuda.stream(other):
            assert kv._stream(None) == other.cuda_stream == kv._stream(other)


@pytest.mark.parametrize("lo,hi", [(0, 24), (40, 256)])
def test_decode_on_cu_masked_stream_is_bit_identical(kv, lo, hi):
    n_cus = torch.cuda.get_device_properties(0).multi_processor_count
    hi = min(hi, n_cus)
    made = cu_masked_stream(lo, hi)
    if made is None:
        pytest.skip("runtime has no hipExtStreamCreateWithCUMask")
    stream, handle = made
    try:
        case = W.thinker_decode(num_sessions=24)
        dp = DevicePool(kv, case.pool.data, 128)
        q, tables, lens = bf16_dev(case.q[0]), i32_dev(case.block_tables), i32_dev(case.context_lens)
        full, ws = _decode(kv, dp, case, q, tables, lens, torch.cuda.current_stream())
        torch.cuda.synchronize()
        for _ in range(2):      # the workspace's counters are reused across grids
            part, _ = _decode(kv, dp, case, q, tables, lens, stream, ws)
            stream.synchronize()
            assert torch.equal(full.view(torch.int16), part.view(torch.int16))
        assert kv.ls_device_errors() == 0
        log("decode on CUs %d..%d bit-identical to the full-device run" % (lo, hi - 1))
    finally:
        torch.cuda.synchronize()
        destroy_stream(handle)


@pytest.mark.parametrize("host", [False, True])
@pytest.mark.parametrize("hq,hkv,d,lens", [
    (32, 4, 128, [9000]), (16, 2, 128, [300, 2500, 1, 1200, 900, 2000]), (32, 4, 128, [700] * 6), (16, 4, 64, [100, 3000, 513]),
    (8, 8, 64, [500, 40, 512])])
def test_small_decode_on_cu_masked_streams(kv, oracle_lib, hq, hkv, d, lens, host):
    """Small batches on streams of 8, 24 and 128 CUs in turn, one workspace: with host lengths the split
    size, and the kernel, follow the stream's CUs at D = 128; with device lengths the bits are those of
    the whole device.  The results are the oracle's on each."""
    rng = np.random.default_rng(len(lens) + d)
    lens = np.array(lens)
    pool, tables, q, _, _ = _synthetic(rng, lens, hq, hkv, d, False)
    dp = DevicePool(kv, pool, d)
    ref = oracle_lib.decode(pool, 16, d, 0, q, tables, lens, 1 / math.sqrt(d))
    ws = torch.full((kv.decode_workspace_bytes(dp.pool, len(lens), hq, tables.shape[1]),), 0x5A, dtype=torch.uint8,
                    device="cuda")
    qd, td, ld = bf16_dev(q), i32_dev(tables), i32_dev(lens)
    full = torch.empty_like(qd)
    kv.paged_attn_decode(dp.pool, 0, qd, td, ld, 1 / math.sqrt(d), full, ws, context_lens_host=lens if host else None)
    assert_attn_close(full, ref, "small decode")
    merges = []
    for hi in (8, 24, 128, 8):
        made = cu_masked_stream(0, hi)
        if made is None:
            pytest.skip("runtime has no hipExtStreamCreateWithCUMask")
        stream, handle = made
        try:
            out = torch.full(q.shape, float("nan"), dtype=torch.bfloat16, device="cuda")
            torch.cuda.synchronize()
            kv.paged_attn_decode(dp.pool, 0, qd, td, ld, 1 / math.sqrt(d), out, ws, stream=stream,
                                 context_lens_host=lens if host else None)
            stream.synchronize()
            assert_attn_close(out, ref, "small decode on %d CUs" % hi)
            if not host:
                assert torch.equal(out.view(torch.int16), full.view(torch.int16)), hi
            merges.append(kv.ls_decode_schedule(dp.pool, len(lens), hq, tables.shape[1], lens if host else None,
                                                stream=stream)["merge"])
        finally:
            torch.cuda.synchronize()
            destroy_stream(handle)
    assert kv.ls_device_errors() == 0
    # 9 to 18 splits of 9000 keys at 4 heads are few on 128 CUs, and too many on 8
    if len(lens) == 1 and host:
        assert not kv.ls_decode_schedule(dp.pool, 1, hq, tables.shape[1], lens)["merge"]
        assert merges[0] and merges[3] and not merges[2]
    if not host:
        assert not any(merges)


def test_split_prefill_on_cu_masked_stream(kv, oracle_lib):
    """A turn whose keys are split by the stream's CUs (24 of them, and 200)."""
    rng = np.random.default_rng(21)
    n, c, d = np.array([150, 20]), np.array([6000, 3000]), 128
    pool, tables, q, kn, vn = _case(rng, n, c, 16, 2, d)
    cu = np.concatenate([[0], np.cumsum(n)]).astype(np.int32)
    ref = oracle_lib.prefill(pool, 16, d, 0, q, kn, vn, cu, c, tables, 1 / math.sqrt(d))
    dp = DevicePool(kv, pool, d)
    args = [bf16_dev(q), i32_dev(cu), i32_dev(c), 150, i32_dev(tables), 1 / math.sqrt(d)]
    new = [bf16_dev(kn), bf16_dev(vn)]
    for lo, hi in ((0, 24), (40, 240)):
        made = cu_masked_stream(lo, hi)
        if made is None:
            pytest.skip("runtime has no hipExtStreamCreateWithCUMask")
        stream, handle = made
        try:
            out = torch.full(q.shape, float("nan"), dtype=torch.bfloat16, device="cuda")
            ws = torch.full((kv.PREFILL_WORKSPACE_BYTES,), 0xFF, dtype=torch.uint8, device="cuda")
            torch.cuda.synchronize()
            kv.paged_attn_prefill(dp.pool, 0, *args, out, *new, lens_host=np.stack([n, c], 1), workspace=ws, stream=stream)
            stream.synchronize()
            assert not bool((ws[kv.PREFILL_COUNTER_BYTES:] == 0xFF).all())        # something was split
            assert_attn_close(out, ref, "split prefill on CUs %d..%d" % (lo, hi - 1))
        finally:
            torch.cuda.synchronize()
            destroy_stream(handle)
    assert kv.ls_device_errors() == 0


def test_restore_on_cu_masked_stream_is_bit_exact(kv):
    made = cu_masked_stream(0, 8)
    if made is None:
        pytest.skip("runtime has no hipExtStreamCreateWithCUMask")
    stream, handle = made
    try:
        rng = np.random.default_rng(11)
        nl, nb, hkv, d = 3, 96, 2, 64
        pool = W.normal_bf16(rng, (nl, nb, 2, hkv, 16 * d))
        dp = DevicePool(kv, pool, d)
        ids = rng.permutation(nb)[:40].astype(np.int32)
        staging = bf16_dev(W.normal_bf16(rng, (40, nl, 2, hkv, 16 * d)))
        kv.kv_blocks_restore(dp.pool, i32_dev(ids), staging, stream=stream)
        stream.synchronize()
        got = dp.host()
        st = host_bits(staging)
        assert np.array_equal(got[:, ids], st.transpose(1, 0, 2, 3, 4))
        others = np.setdiff1d(np.arange(nb), ids)
        assert np.array_equal(got[:, others], pool[:, others])
        back = torch.empty_like(staging)
        kv.kv_blocks_stash(dp.pool, i32_dev(ids), back, stream=stream)
        stream.synchronize()
        assert torch.equal(back.view(torch.int16), staging.view(torch.int16))
        assert kv.ls_device_errors() == 0
    finally:
        torch.cuda.synchronize()
        destroy_stream(handle)
