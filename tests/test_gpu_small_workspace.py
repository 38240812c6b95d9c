"""The rejection half alone on a workspace that holds the records of few blocks only (what the size query
of another batch may have given): it runs on fewer blocks, stays inside the workspace and agrees with the oracle."""
import numpy as np
import pytest

from paper_2406_14066_amd import spec_verify as sv
from paper_2406_14066_amd import workloads as W
from parity_utils import check_reject
from test_reject_plan_host import small_records

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,k,V", [(8, 4, 128256), (15, 8, 128256), (33, 2, 40004)])
def test_few_records(B, k, V):
    import torch
    from paper_2406_14066_amd import harness as H
    print("case small workspace", B, k, V, flush=True)
    w = W.make_workload("few", B=B, Hq=1, Hkv=1, d=64, V=V, dtype="f32", kv_len=[16] * B, k=[k] * B, draft_std=3.0,
                        sigma=0.8, data_seed=B, philox_seed=17, with_kv=False)
    w.k_pages = w.v_pages = np.zeros((1, 1, 16, 64), np.float32)
    w.q = np.zeros((w.T, 1, 64), np.float32)
    ds = H.DeviceStep(w, kv_layout=sv.KV_TOKEN_MAJOR)
    need = small_records(B, k, V)
    assert need < sv.spec_verify_workspace_bytes(None, ds.reject_args)
    buffer = sv.alloc_workspace(need + 4096)
    buffer.fill_(0x5A)
    ds.workspace = buffer[:need]
    for _ in range(2):
        ds.counters.zero_()
        ds.out_tokens.fill_(-7)
        ds.run_reject()
        check_reject(w, ds.results(), max_excluded=1)
    assert bool((buffer[need:] == 0x5A).all())
    ds.workspace = buffer[: need - 256]
    with pytest.raises(Exception, match="too small"):
        ds.run_reject()
    torch.cuda.synchronize()
