"""The whole step captured into a HIP graph and replayed (Section 5.3 of the paper runs its
steps from captured graphs): the library allocates nothing, clears nothing with memsets and
tags its workspace records per call, so a captured launch must give the eager result on
every replay, with the program's own eager work in between."""
import numpy as np
import pytest

from paper_2406_14066_amd import workloads as W
from paper_2406_14066_amd import spec_verify as sv
from parity_utils import check_attn, check_reject

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("name,kw,early_stop", [("c2", dict(B=4, L_scale=0.25), False),
                                                ("c4", dict(B=40, L_scale=0.5, V=8192), False),
                                                ("c4", dict(B=40, L_scale=0.5, V=8192), True),
                                                ("c5", dict(L_scale=0.1, V=16384), False)],
                         ids=["c2_small", "c4_small", "c4_small_early_stop", "c5_small"])
def test_step_replays_from_a_graph(tuning, name, kw, early_stop):
    import torch
    from paper_2406_14066_amd.harness import DeviceStep
    print("case graph", name, "early stop", early_stop, flush=True)
    if early_stop:   # the statistics pass in position order with placeholder records (large batches get it by themselves)
        tuning("SPEC_VERIFY_EARLY_STOP", 1)
    w = W.config(name, **kw)
    ds = DeviceStep(w, kv_layout=sv.KV_MFMA)
    ds.run_step()
    eager = ds.results()
    check_attn(w, eager["out"])
    check_reject(w, eager)

    graph = torch.cuda.CUDAGraph()
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        ds.run_step(side)          # warm-up on the capture stream
    torch.cuda.synchronize()
    with torch.cuda.graph(graph, stream=side):
        ds.run_step(torch.cuda.current_stream())
    torch.cuda.synchronize()

    scratch = torch.zeros(1 << 20, device="cuda")
    for replay in range(5):
        # the program's own eager work between the replays, and outputs reset to a sentinel
        ds.out.fill_(float("nan"))
        ds.accepted_len.fill_(-9)
        ds.next_token.fill_(-9)
        ds.out_tokens.fill_(-9)
        ds.counters.zero_()
        scratch.add_(1.0)
        if replay == 2:
            ds.run_step()           # an eager call on the same workspace between two replays
            ds.counters.zero_()
        torch.cuda.synchronize()
        graph.replay()
        got = ds.results()
        np.testing.assert_array_equal(got["out"], eager["out"])
        np.testing.assert_array_equal(got["accepted_len"], eager["accepted_len"])
        np.testing.assert_array_equal(got["next_token"], eager["next_token"])
        np.testing.assert_array_equal(got["out_tokens"], eager["out_tokens"])
        np.testing.assert_array_equal(got["counters"], eager["counters"])


# a replayed launch reuses its tickets' tag: a replay in which a request has outgrown what the chunks that the launch lists can hold leaves nothing behind
# that the next one, with lengths that fit again, would take for its own
def test_replay_after_one_whose_lengths_did_not_fit(tuning):
    import torch
    from paper_2406_14066_amd.harness import DeviceStep
    print("case graph outgrown", flush=True)
    kv_len = (4000, 600, 64, 6000)
    w = W.make_workload("outgrown", B=len(kv_len), Hq=16, Hkv=16, d=128, V=256, dtype="bf16", kv_len=list(kv_len), k=[2] * 4, draft_std=2.0,
                        sigma=0.8, data_seed=3, philox_seed=9)
    w.block_table = np.concatenate([w.block_table, w.block_table], axis=1)   # room for the longer lengths (any pages will do)
    ds = DeviceStep(w, kv_layout=sv.KV_TOKEN_MAJOR)
    plan = sv.spec_verify_plan(ds.attn_args, None)
    C = plan["chunk_tokens"]
    assert plan["attn_blocks"] == 16 * sum(-(-n // C) for n in kv_len) < 16 * len(kv_len) * plan["max_chunks"] and C < 4096 < C * plan["max_chunks"], plan
    errors = torch.zeros(1, dtype=torch.int64, device="cuda")
    ds.attn_args.error_count = errors.data_ptr()
    good = ds.kv_len.clone()
    long = good.clone()
    long[2] = 4097      # one chunk is listed, and no chunk has more than 4096 tokens
    graph, side = torch.cuda.CUDAGraph(), torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        ds.run_attn(side)
    torch.cuda.synchronize()
    eager = ds.out.cpu().numpy()
    check_attn(w, eager)
    with torch.cuda.graph(graph, stream=side):
        ds.run_attn(torch.cuda.current_stream())
    torch.cuda.synchronize()
    for lens, found in ((good, 0), (long, 1), (good, 0), (long, 1), (long, 1), (good, 0), (good, 0)):
        ds.kv_len.copy_(lens)
        ds.out.fill_(float("nan"))
        errors.zero_()
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert int(errors.item()) == found
        got = ds.out.cpu().numpy()
        rows = slice(int(w.cu_q_len[2]), int(w.cu_q_len[3]))
        if found:
            assert np.isnan(got[rows]).all()
            got[rows] = eager[rows]
        np.testing.assert_array_equal(got, eager)


# the early stop that looks at what its request's earlier positions have published, replayed: every replay draws other random numbers, so that
# a record left from the one before would show another rejection.  One row tile, the rejection half first; two row tiles and wave
# groups in the mixed order of the grid (more blocks of each half than go first).
@pytest.mark.parametrize("ragged", [False, True], ids=["uniform", "ragged"])
@pytest.mark.parametrize("B,Hq,Hkv,k,V,mixed", [(64, 2, 1, 6, 2052, False), (80, 32, 8, 7, 8192, True), (80, 64, 8, 7, 8192, True)])
def test_looking_early_stop_replays_from_a_graph(tuning, B, Hq, Hkv, k, V, mixed, ragged):
    import torch
    from paper_2406_14066_amd.harness import DeviceStep
    print("case graph look", B, Hq, Hkv, k, V, ragged, flush=True)
    tuning("SPEC_VERIFY_EARLY_STOP", 2)
    ks = np.random.default_rng(B).integers(2, k + 1, size=B) if ragged else np.full(B, k)
    ks[0] = k
    w = W.make_workload("look_graph", B=B, Hq=Hq, Hkv=Hkv, d=128, V=V, dtype="bf16", kv_len=[40 + b for b in range(B)], k=ks, draft_std=3.0,
                        sigma=0.8, data_seed=B, philox_seed=5)
    ds = DeviceStep(w, kv_layout=sv.KV_TOKEN_MAJOR)
    step = torch.zeros(1, dtype=torch.int64, device="cuda")
    ds.reject_args.philox_step_device = step.data_ptr()
    plan = ds.plan()
    assert plan["early_stop"] == 1 and mixed == (plan["attn_blocks"] > 512 and plan["reject_blocks"] > 1024), plan
    assert (plan["row_tiles"], plan["row_groups"]) == {2: (1, 1), 32: (2, 1), 64: (2, 2)}[Hq], plan
    graph, side = torch.cuda.CUDAGraph(), torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        ds.run_step(side)
    torch.cuda.synchronize()
    with torch.cuda.graph(graph, stream=side):
        ds.run_step(torch.cuda.current_stream())
    torch.cuda.synchronize()
    out = None
    for replay in range(4):
        w.philox_step = 1000 + replay
        step.fill_(w.philox_step)
        ds.out.fill_(float("nan"))
        for t in (ds.accepted_len, ds.next_token, ds.out_tokens):
            t.fill_(-9)
        ds.counters.zero_()
        torch.cuda.synchronize()
        graph.replay()
        got = ds.results()
        check_reject(w, got, max_excluded=1)
        if out is None:
            check_attn(w, got["out"])
            out = got["out"]
        np.testing.assert_array_equal(got["out"], out)
