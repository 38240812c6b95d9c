"""How the planner splits the rejection half (host only: plans are made without a GPU)."""
import numpy as np
import pytest

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


# long race segments beside a short attention half end the launch: at least as many as 512 blocks give
@pytest.mark.parametrize("B,k,length,V,least", [(128, 1, 400, 64128, 4), (256, 1, 400, 64128, 2), (64, 1, 400, 128256, 8),
                                                (128, 1, 400, 128256, 4), (64, 4, 1000, 128256, 8)])
def test_large_vocabulary_beside_a_short_attention_half(B, k, length, V, least):
    assert step_plan(B, k, length, V)["race_segments"] >= least


# where the segments are short, or the launch long, few blocks hold the attention's slots
@pytest.mark.parametrize("B,k,length,V,segments", [(256, 2, 640, 32000, 1), (64, 1, 400, 32000, 4), (24, 4, 2000, 128256, 11),
                                                   (128, 4, 400, 32000, 2)])
def test_few_race_blocks_beside_a_long_attention_half(B, k, length, V, segments):
    assert step_plan(B, k, length, V)["race_segments"] == segments
