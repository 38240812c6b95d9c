"""Sizes at which the rejection half's stages can go wrong, against the CPU oracle: the edges of the
batches in which a block streams a logit row, and equal maxima wherever they can sit."""
import numpy as np
import pytest

import oracle
from paper_2406_14066_amd import workloads as W
from paper_2406_14066_amd import spec_verify as sv
from parity_utils import check_reject

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def harness():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_2406_14066_amd import harness as H
    return H


def _logits_only(B, V, k, seed):
    w = W.make_workload("stages", B=B, Hq=1, Hkv=1, d=64, V=V, dtype="f32", kv_len=[16] * B, k=k, draft_std=3.0,
                        sigma=0.8, data_seed=seed, philox_seed=99 + seed, with_kv=False)
    w.k_pages = w.v_pages = np.zeros((1, 1, 16, 64), np.float32)
    w.q = np.zeros((w.T, 1, 64), np.float32)
    return w


# a batch of the streaming pass is 4096 logits, a ring of them 16384; a row is cut into segments of 8192 or more
@pytest.mark.parametrize("V", [4, 1020, 4092, 4096, 4100, 16380, 16388, 20484, 65540], ids=lambda v: "V%d" % v)
def test_streamed_rows_at_batch_edges(harness, V):
    print("case stream edges", V, flush=True)
    k = [3, 0, 5, 1]
    w = _logits_only(4, V, k, seed=V)
    ds = harness.DeviceStep(w, kv_layout=sv.KV_TOKEN_MAJOR)
    ds.run_reject()
    check_reject(w, ds.results())

    # greedy: integer logits (many equal maxima), a maximum in the last and in a middle place, a row of -inf
    w.target_logits = np.round(np.clip(w.target_logits, -6, 6)).astype(np.float32)
    w.target_logits[1, [V - 1, V // 2]] = 9.0
    w.target_logits[2] = -np.inf
    w.target_logits[3, V - 1] = 9.0
    for b in range(w.B):
        t0 = int(w.cu_q_len[b])
        for i in range(k[b]):
            w.draft_tokens[t0 - b + i] = int(np.argmax(w.target_logits[t0 + i]))   # (the first of equal maxima)
    ref = oracle.reject_greedy(w.target_logits, w.draft_tokens, w.cu_q_len)
    ds = harness.DeviceStep(w, kv_layout=sv.KV_TOKEN_MAJOR, accept_mode=sv.ACCEPT_GREEDY)
    ds.run_reject()
    res = ds.results()
    for name in ("accepted_len", "next_token", "out_tokens", "counters"):
        np.testing.assert_array_equal(res[name], getattr(ref, name))
    assert (ref.accepted_len == k).all()


# a race block takes 1024 ids at a time and parts of 8192; one segment per request makes the last part ragged
@pytest.mark.parametrize("mode", [sv.ACCEPT_SAMPLE, sv.ACCEPT_POINT_DRAFT], ids=["sample", "point"])
@pytest.mark.parametrize("V", [4, 1024, 1028, 8188, 8196, 20484], ids=lambda v: "V%d" % v)
def test_race_of_one_segment_at_part_edges(harness, tuning, V, mode):
    print("case race parts", V, mode, flush=True)
    tuning("SPEC_VERIFY_RACE_BLOCKS", 1)
    w = _logits_only(5, V, [2, 0, 8, 1, 4], seed=V + 1)
    ds = harness.DeviceStep(w, kv_layout=sv.KV_TOKEN_MAJOR, accept_mode=mode)
    assert ds.plan()["race_segments"] == 1
    ds.run_reject()
    ref = None
    if mode == sv.ACCEPT_POINT_DRAFT:
        ref = oracle.reject_onehot(w.target_logits, w.draft_tokens, w.cu_q_len, w.philox_seed, w.philox_step)
    check_reject(w, ds.results(), ref=ref)


# the final stage takes 1, 2, 4, 8 or 16 requests per block, depending on their number
@pytest.mark.parametrize("mode", [sv.ACCEPT_SAMPLE, sv.ACCEPT_GREEDY, sv.ACCEPT_POINT_DRAFT], ids=["sample", "greedy", "point"])
@pytest.mark.parametrize("B", [1, 15, 16, 33, 67, 131], ids=lambda b: "B%d" % b)
def test_requests_grouped_in_the_final_stage(harness, B, mode):
    print("case final groups", B, mode, flush=True)
    rng = np.random.default_rng(B)
    w = _logits_only(B, 2052, rng.integers(0, 9, size=B), seed=B)
    if mode == sv.ACCEPT_GREEDY:
        hit = rng.random(w.T - B) < 0.7
        rows = np.concatenate([np.arange(w.cu_q_len[b], w.cu_q_len[b + 1] - 1) for b in range(B)])
        w.draft_tokens = np.where(hit, w.target_logits[rows].argmax(1), w.draft_tokens).astype(np.int32)
    ds = harness.DeviceStep(w, kv_layout=sv.KV_TOKEN_MAJOR, accept_mode=mode)
    for _ in range(2):   # the second call finds the first one's records cleared or out of date
        ds.counters.zero_()
        ds.out_tokens.fill_(-7)
        ds.run_reject()
        res = ds.results()
        if mode == sv.ACCEPT_GREEDY:
            ref = oracle.reject_greedy(w.target_logits, w.draft_tokens, w.cu_q_len)
            for name in ("accepted_len", "next_token", "out_tokens", "counters"):
                np.testing.assert_array_equal(res[name], getattr(ref, name))
        else:
            ref = None
            if mode == sv.ACCEPT_POINT_DRAFT:
                ref = oracle.reject_onehot(w.target_logits, w.draft_tokens, w.cu_q_len, w.philox_seed, w.philox_step)
            check_reject(w, res, ref=ref, max_excluded=1)


# rows in position order, each skipped if what its request's earlier positions have published shows a rejection: one draft
# length and several, one block's worth of requests and (several lengths, which then keep the request order) more
@pytest.mark.parametrize("mode", [sv.ACCEPT_SAMPLE, sv.ACCEPT_GREEDY, sv.ACCEPT_POINT_DRAFT], ids=["sample", "greedy", "point"])
@pytest.mark.parametrize("B,V,uniform", [(1, 1024, True), (1, 70000, False), (63, 2052, False), (64, 2052, True), (129, 17000, False),
                                         (256, 2052, False), (257, 2052, False), (300, 1024, True)],
                         ids=lambda v: str(v))
def test_early_stop_that_looks_at_earlier_positions(harness, tuning, B, V, uniform, mode):
    print("case look", B, V, uniform, mode, flush=True)
    rng = np.random.default_rng(B + V)
    w = W.make_workload("look", B=B, Hq=1, Hkv=1, d=64, V=V, dtype="bf16", kv_len=[16] * B, k=[6] * B if uniform else rng.integers(0, 9, size=B),
                        draft_std=3.0, sigma=0.8, data_seed=B, philox_seed=99 + B)
    if mode == sv.ACCEPT_GREEDY:
        hit = rng.random(w.T - B) < 0.7
        rows = np.concatenate([np.arange(w.cu_q_len[b], w.cu_q_len[b + 1] - 1) for b in range(B)])
        w.draft_tokens = np.where(hit, w.target_logits[rows].argmax(1), w.draft_tokens).astype(np.int32)
    tuning("SPEC_VERIFY_EARLY_STOP", 2)
    ds = harness.DeviceStep(w, kv_layout=sv.KV_TOKEN_MAJOR, accept_mode=mode)
    assert ds.plan()["early_stop"] == (1 if w.T > B and (uniform or B <= 256) else 0)
    for _ in range(2):   # the second call finds the first one's records cleared or out of date
        ds.counters.zero_()
        ds.out_tokens.fill_(-7)
        ds.run_step()
        res = ds.results()
        if mode == sv.ACCEPT_GREEDY:
            ref = oracle.reject_greedy(w.target_logits, w.draft_tokens, w.cu_q_len)
            for name in ("accepted_len", "next_token", "out_tokens", "counters"):
                np.testing.assert_array_equal(res[name], getattr(ref, name))
        else:
            ref = None
            if mode == sv.ACCEPT_POINT_DRAFT:
                ref = oracle.reject_onehot(w.target_logits, w.draft_tokens, w.cu_q_len, w.philox_seed, w.philox_step)
            check_reject(w, res, ref=ref, max_excluded=1)


# ... and rows are skipped, none but those after a request's first rejection.  The final stage clears the records of the requests that it
# serves; with one poll per wait it abandons most of them, and theirs stay behind in the workspace.
@pytest.mark.parametrize("mode", [sv.ACCEPT_SAMPLE, sv.ACCEPT_GREEDY, sv.ACCEPT_POINT_DRAFT], ids=["sample", "greedy", "point"])
@pytest.mark.parametrize("B,uniform", [(300, True), (256, False)], ids=["uniform", "ragged"])
def test_early_stop_that_looks_skips_rows(harness, tuning, B, uniform, mode):
    print("case skipped rows", B, uniform, mode, flush=True)
    rng = np.random.default_rng(B)
    w = W.make_workload("skip", B=B, Hq=1, Hkv=1, d=64, V=1024, dtype="bf16", kv_len=[16] * B, k=[8] * B if uniform else rng.integers(4, 9, size=B),
                        draft_std=3.0, sigma=0.8, data_seed=B, philox_seed=7)
    if mode == sv.ACCEPT_SAMPLE:
        ref = oracle.reject_sample(w.target_logits, w.draft_logits, w.draft_tokens, w.cu_q_len, w.philox_seed, w.philox_step)
    elif mode == sv.ACCEPT_GREEDY:
        ref = oracle.reject_greedy(w.target_logits, w.draft_tokens, w.cu_q_len)
    else:
        ref = oracle.reject_onehot(w.target_logits, w.draft_tokens, w.cu_q_len, w.philox_seed, w.philox_step)
    after = np.zeros(2 * w.T - w.B, dtype=bool)       # rows after a first rejection: target rows, then draft rows
    for b in range(B):
        t0, t1, m = int(w.cu_q_len[b]), int(w.cu_q_len[b + 1]), int(ref.accepted_len[b])
        after[t0 + m + 1: t1] = True
        after[w.T + t0 - b + m + 1: w.T + t1 - b - 1] = True
    tuning("SPEC_VERIFY_EARLY_STOP", 2)
    tuning("SPEC_VERIFY_SPIN_LIMIT", 1)
    ds = harness.DeviceStep(w, kv_layout=sv.KV_TOKEN_MAJOR, accept_mode=mode)
    plan = ds.plan()
    assert plan["early_stop"] == 1 and plan["stat_segments"] == 1, plan
    ds.workspace.zero_()
    ds.run_step()
    gone = ds.results()["accepted_len"] < 0
    base = sv.spec_verify_workspace_bytes(ds.attn_args, None)
    rows = w.T if mode != sv.ACCEPT_SAMPLE else len(after)
    rec = ds.workspace.cpu().numpy().view(np.uint8)[base: base + rows * 24].view(np.uint32).reshape(rows, 3, 2)   # (value, tag) of three words
    # a skipped row's record: the largest logit of nothing, or a sum of 1 at offset 0
    value = (0xFF800000, 0x7FFFFFFF) if mode == sv.ACCEPT_GREEDY else (0, 0x3FF00000, 0)
    skipped = (rec[:, 0, 1] != 0) & np.all(rec[:, : len(value), 0] == np.array(value, dtype=np.uint32), axis=1)
    print("abandoned %d of %d requests, rows after a rejection %d, skipped among what is left %d" % (gone.sum(), B, after[:rows].sum(), skipped.sum()),
          flush=True)
    assert gone.any() and skipped.any() and not (skipped & ~after[:rows]).any()


def test_offsets_far_apart_and_segments_of_nothing(harness):
    """Row statistics whose segments differ by thousands of powers of two, and segments of nothing but -inf: the
    accept chain rescales them exactly (a segment far below the row's maximum adds nothing)."""
    print("case far offsets", flush=True)
    w = _logits_only(3, 32768, [4, 2, 8], seed=3)
    V = w.V
    w.target_logits[:, : V // 4] -= 3000.0
    w.draft_logits[:, : V // 4] -= 3000.0
    w.target_logits[:, V // 4: V // 2] = -np.inf
    w.draft_logits[:, V // 4: V // 2] = -np.inf
    rng = np.random.default_rng(0)
    w.draft_tokens = rng.integers(V // 2, V, size=w.T - w.B).astype(np.int32)
    ds = harness.DeviceStep(w, kv_layout=sv.KV_TOKEN_MAJOR)
    assert ds.plan()["stat_segments"] >= 4
    ds.run_reject()
    check_reject(w, ds.results())
