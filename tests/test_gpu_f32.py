"""The fp32 step kernel against the CPU oracle and the scalar kernels: every number of row tiles and wave
groups, both head dims, lengths around pages and chunks, split requests, a length bucket, and values that
are not finite where a query cannot see them."""
import numpy as np
import pytest

import oracle
from paper_2406_14066_amd import workloads as W
from paper_2406_14066_amd import spec_verify as sv
from parity_utils import check_attn, check_reject

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def harness():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_2406_14066_amd import harness as H
    return H


def _workload(Hq, Hkv, d, kv_len, k, seed):
    return W.make_workload("f32", B=len(kv_len), Hq=Hq, Hkv=Hkv, d=d, V=1028, dtype="f32", kv_len=kv_len, k=k,
                           draft_std=2.0, sigma=0.8, data_seed=seed, philox_seed=seed)


# fused rows per KV head: 1, 16, 18, 32, 33, 64, 65, 128, 144
@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("Hq,Hkv,kmax", [(3, 3, 0), (4, 1, 3), (4, 2, 8), (8, 2, 7), (33, 3, 2), (16, 2, 7), (13, 1, 4), (32, 2, 7), (16, 1, 8)])
def test_rows_and_lengths(harness, Hq, Hkv, kmax, d):
    print("case f32 rows", Hq, Hkv, kmax, d, flush=True)
    k = [kmax, 0, kmax // 2, kmax, kmax]
    w = _workload(Hq, Hkv, d, [kmax + 1, 17, 64 + kmax, 300, 1111], k, seed=Hq * 10 + d)
    ds = harness.DeviceStep(w)
    assert ds.plan()["launches"] == 1
    ds.run_step()
    res = ds.results()
    check_attn(w, res["out"])
    check_reject(w, res)
    ds.out.zero_()
    ds.run_attn()
    np.testing.assert_array_equal(ds.results()["out"], res["out"])


# 64 dims beside a race and more rejection blocks than block slots: K with the streaming hint up to a longest request of 1536 tokens.  The hint
# changes no result: the attention alone, which runs without it, gives the same bits
@pytest.mark.parametrize("longest", [1536, 1537])
@pytest.mark.parametrize("Hq,Hkv,k,tiles", [(4, 2, 6, 1), (8, 2, 7, 2)])
def test_k_with_the_streaming_hint(harness, tuning, Hq, Hkv, k, tiles, longest):
    print("case f32 K hint", Hq, Hkv, k, longest, flush=True)
    tuning("SPEC_VERIFY_F32_SCALAR", 0)
    B = 150
    kv_len = [longest if b == 70 else k + 1 + (37 * b) % 90 for b in range(B)]
    w = _workload(Hq, Hkv, 64, kv_len, [k] * B, seed=tiles)
    ds = harness.DeviceStep(w)
    plan = ds.plan()
    assert plan["reject_blocks"] > 1024 and (plan["row_tiles"], plan["row_groups"]) == (tiles, 1), plan
    ds.run_step()
    res = ds.results()
    check_attn(w, res["out"])
    check_reject(w, res, max_excluded=1)
    if sv.spec_verify_plan(ds.attn_args, None)["chunk_tokens"] == plan["chunk_tokens"]:
        ds.out.zero_()
        ds.run_attn()
        np.testing.assert_array_equal(ds.results()["out"], res["out"])


@pytest.mark.parametrize("bucket", [0, 2048])
@pytest.mark.parametrize("chunk", [16, 48, 1024])
def test_split_requests(harness, tuning, chunk, bucket):
    print("case f32 split", chunk, bucket, flush=True)
    w = _workload(8, 4, 128, [9, 1030, 515, 100], [4, 8, 1, 0], seed=chunk)
    tuning("SPEC_VERIFY_CHUNK", chunk)
    if bucket:
        w.block_table = np.pad(w.block_table, ((0, 0), (0, bucket // 16 - w.block_table.shape[1])))
    ds = harness.DeviceStep(w, max_kv_len=bucket)
    ds.run_step()
    res = ds.results()
    check_attn(w, res["out"])
    check_reject(w, res)


@pytest.mark.parametrize("poison", [np.nan, np.inf, -np.inf], ids=["nan", "plus_inf", "minus_inf"])
@pytest.mark.parametrize("Hq,Hkv", [(2, 2), (8, 1), (16, 1)])
def test_values_a_query_cannot_see(harness, tuning, Hq, Hkv, poison):
    """The K and V rows of the later draft positions, and every slot past the end, hold `poison`: the rows
    that see none of it come out as they do without it, and the others as from the scalar kernels."""
    print("case f32 poison", Hq, poison, flush=True)
    w = _workload(Hq, Hkv, 128, [37, 260, 21], [4, 8, 3], seed=7)
    clean = oracle.verify_attn(w.q, w.k_pages, w.v_pages, w.block_table, w.kv_len, w.cu_q_len)
    for pool in (w.k_pages, w.v_pages):
        pool[(pool == np.float32(W.FILLER)).all(axis=-1)] = poison
    sees = np.zeros(w.T, dtype=bool)
    for b in range(w.B):
        last = int(w.kv_len[b]) - 1          # the two last draft positions
        for t in (last - 1, last):
            w.k_pages[w.block_table[b, t // 16], :, t % 16] = poison
            w.v_pages[w.block_table[b, t // 16], :, t % 16] = poison
        sees[int(w.cu_q_len[b + 1]) - 2: int(w.cu_q_len[b + 1])] = True
    ds = harness.DeviceStep(w)
    ds.run_attn()
    got = ds.results()["out"]
    np.testing.assert_allclose(got[~sees], clean[~sees], rtol=0, atol=1e-5)
    tuning("SPEC_VERIFY_FORCE_GENERIC", 1)
    ds = harness.DeviceStep(w)
    ds.run_attn()
    want = ds.results()["out"]
    np.testing.assert_allclose(got, want, rtol=0, atol=1e-5)
    assert np.isnan(want[sees]).any()
