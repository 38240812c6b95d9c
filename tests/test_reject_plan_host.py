"""How the planner splits the rejection half (host only: plans are made without a GPU)."""
import ctypes as C

import numpy as np
import pytest
import torch

from paper_2406_14066_amd import spec_verify as sv

FAKE = 0x1000  # non-null, aligned, never dereferenced


def attn_args(B, k, length, Hq=64, Hkv=8, d=128, dtype=sv.SPEC_BF16, layout=sv.KV_MFMA, q_len=None):
    hc = np.concatenate([[0], np.cumsum(q_len if q_len is not None else [k + 1] * B)]).astype(np.int32)
    hk = np.full(B, length, dtype=np.int32)
    a = sv.AttnArgs()
    a.B, a.Hq, a.Hkv, a.d = B, Hq, Hkv, d
    a.block_size, a.num_blocks, a.max_blocks_per_req = 16, 1 << 20, (length + 15) // 16
    a.T, a.qkv_dtype, a.kv_layout = int(hc[-1]), dtype, layout
    for f in ("q", "k_cache", "v_cache", "block_table", "kv_len", "cu_q_len", "out"):
        setattr(a, f, FAKE)
    a.host_kv_len, a.host_cu_q_len, a._keep = hk.ctypes.data, hc.ctypes.data, (hk, hc)
    return a


def reject_args(B, k, V, mode=sv.ACCEPT_SAMPLE, q_len=None):
    hc = np.concatenate([[0], np.cumsum(q_len if q_len is not None else [k + 1] * B)]).astype(np.int32)
    r = sv.RejectArgs()
    r.B, r.V, r.T, r.accept_mode = B, V, int(hc[-1]), mode
    for f in ("target_logits", "draft_logits", "draft_tokens", "cu_q_len", "accepted_len", "next_token", "counters"):
        setattr(r, f, FAKE)
    r.host_cu_q_len, r._keep = hc.ctypes.data, (hc,)
    return r


def step_plan(B, k, length, V, **kw):
    return sv.spec_verify_plan(attn_args(B, k, length, **kw), reject_args(B, k, V))


# long race segments beside a short attention half end the launch: as many as 512 blocks give (384 where the attention goes first)
@pytest.mark.parametrize("B,k,length,V,least", [(128, 1, 400, 64128, 4), (256, 1, 400, 64128, 2), (64, 1, 400, 128256, 6),
                                                (128, 1, 400, 128256, 4), (64, 4, 1000, 128256, 6), (128, 4, 400, 64128, 3)])
def test_large_vocabulary_beside_a_short_attention_half(B, k, length, V, least):
    assert step_plan(B, k, length, V)["race_segments"] >= least


# where the segments are short, or the launch long, few blocks hold the attention's slots
@pytest.mark.parametrize("B,k,length,V,segments", [(256, 2, 640, 32000, 1), (64, 1, 400, 32000, 4), (24, 4, 2000, 128256, 11), (48, 4, 150, 128256, 6),
                                                   (128, 4, 400, 32000, 2)])
def test_few_race_blocks_beside_a_long_attention_half(B, k, length, V, segments):
    assert step_plan(B, k, length, V)["race_segments"] == segments


# beside an attention half, long drafts and draft lengths of their own stop early where that saves enough rows; not alone, nor
# with draft lengths of more requests than a block has threads
@pytest.mark.parametrize("B,k,length,V,ragged,stops", [(96, 7, 640, 32000, False, 1), (200, 3, 400, 32000, True, 1), (256, 8, 200, 17000, True, 1), (255, 8, 52, 8016, True, 0),
                                                       (257, 8, 200, 17000, True, 0), (64, 5, 580, 32000, True, 0), (8, 4, 2048, 32000, False, 0)])
def test_early_stop_beside_an_attention_half(B, k, length, V, ragged, stops):
    q_len = [1 + (1 + b % k) for b in range(B)] if ragged else None
    r = reject_args(B, k, V, q_len=q_len)
    assert sv.spec_verify_plan(attn_args(B, k, length, q_len=q_len), r)["early_stop"] == stops
    if ragged:
        assert sv.spec_verify_plan(None, r)["early_stop"] == 0


# chunks sized from all lengths: the launch has the blocks that the rejection half's plan counts on, one per chunk that exists
@pytest.mark.parametrize("lens,V", [([8000] * 3 + [1000] * 13, 32000), ([16000] * 2 + [500] * 14, 32000), ([32000] + [800] * 7, 32000),
                                    ([8000] * 2 + [300] * 14, None), ([12000] + [400] * 15, None)])
def test_listed_chunks_are_the_blocks_of_the_launch(lens, V):
    a = attn_args(len(lens), 3, max(lens), Hq=32)
    hk = np.asarray(lens, dtype=np.int32)
    a.host_kv_len, a._keep = hk.ctypes.data, a._keep + (hk,)
    plan = sv.spec_verify_plan(a, None if V is None else reject_args(len(lens), 3, V))
    assert plan["attn_blocks"] == 8 * sum((n + plan["chunk_tokens"] - 1) // plan["chunk_tokens"] for n in lens) <= 256


# beside a short attention half whose rejection blocks fill the chip and go first, an eighth of the units is left to them
@pytest.mark.parametrize("lens,k,V,Hq,blocks", [([60 + 850 * i for i in range(8)], 2, 128256, 64, 224), ([6000] * 3 + [900] * 9, 1, 128256, 32, 224),
                                                ([200 + 300 * i for i in range(17)], 1, 8192, 32, 256), ([200 + 1000 * i for i in range(11)], 4, 32000, 32, 256)])
def test_listed_chunks_beside_rejection_blocks_that_go_first(lens, k, V, Hq, blocks):
    a = attn_args(len(lens), k, max(lens), Hq=Hq)
    hk = np.asarray(lens, dtype=np.int32)
    a.host_kv_len, a._keep = hk.ctypes.data, a._keep + (hk,)
    plan = sv.spec_verify_plan(a, reject_args(len(lens), k, V))
    assert plan["attn_blocks"] == 8 * sum((n + plan["chunk_tokens"] - 1) // plan["chunk_tokens"] for n in lens)
    assert blocks - 32 < plan["attn_blocks"] <= blocks, plan


def small_records(B, k, V, mode=sv.ACCEPT_SAMPLE):
    """Bytes of the rejection half's records with about 256 statistics and 512 race blocks: the least that
    the half alone works with."""
    rows = (2 * k + 1) * B if mode == sv.ACCEPT_SAMPLE else (k + 1) * B

    def split(blocks, n, least, most):
        segs = max(1, min((blocks + n - 1) // n, (V + least - 1) // least, most))
        length = ((V + segs - 1) // segs + 3) // 4 * 4
        return (V + length - 1) // length

    def align(n):
        return (n + 255) // 256 * 256

    return align(24 * rows * split(256, rows, 8192, 32)) + align(8 * (2 * B * split(512, B, 2048, 64) + B))


@pytest.mark.parametrize("mode", [sv.ACCEPT_SAMPLE, sv.ACCEPT_GREEDY, sv.ACCEPT_POINT_DRAFT])
@pytest.mark.parametrize("V", [1024, 32000, 128256])
def test_a_workspace_for_the_largest_batch_serves_every_smaller_one(V, mode):
    largest = {}
    for B in list(range(1, 66)) + [96, 127, 128, 255, 256, 600, 1500]:
        for k in range(0, 9):
            largest[B, k] = sv.spec_verify_workspace_bytes(None, reject_args(B, k, V, mode))
            assert largest[B, k] >= small_records(B, k, V, mode)
            if k > 0:
                assert largest[B, k] >= largest[B, k - 1], (B, k)
        if B > 1:
            before = max(b for b, _ in largest if b < B)
            assert all(largest[B, k] >= largest[before, k] for k in range(0, 9)), B
    # ... and so does the workspace of a step of the largest batch
    step = sv.spec_verify_workspace_bytes(attn_args(64, 8, 300), _with_mode(reject_args(64, 8, V), mode))
    assert step >= largest[64, 8]


def _with_mode(r, mode):
    r.accept_mode = mode
    return r


@pytest.mark.skipif(torch.cuda.is_available(), reason="the pointers of this test are not real")
def test_a_workspace_without_room_for_many_blocks_is_not_refused():
    for B in (1, 4, 15, 16, 33, 64, 200):
        for k in (0, 1, 4, 8):
            for V in (1024, 32000, 128256):
                r, need = reject_args(B, k, V), small_records(B, k, V)
                call = lambda n: sv.lib().spec_reject_sample(C.byref(r), FAKE, n, None)
                # (no GPU here: past the size check the launch fails)
                assert call(need) == sv.SPEC_EHIP, (B, k, V)
                assert call(need - 256) == sv.SPEC_EWORKSPACE, (B, k, V)


# the early stop's chain beside an attention half whose blocks all go first in the grid: measured slower in every case
@pytest.mark.parametrize("B,k,length,V", [(64, 1, 1000, 32000), (64, 2, 1000, 8192), (64, 1, 1000, 128256), (32, 1, 1024, 8192)])
def test_no_early_stop_beside_attention_blocks_that_go_first(B, k, length, V):
    assert step_plan(B, k, length, V)["early_stop"] == 0


@pytest.mark.parametrize("B,k,length,V", [(256, 2, 640, 32000), (128, 4, 512, 32000), (256, 1, 400, 64128)])
def test_early_stop_beside_many_attention_blocks(B, k, length, V):
    assert step_plan(B, k, length, V)["early_stop"] == 1
