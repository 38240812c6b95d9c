"""Which kernel an fp32 attention call takes, and that a workspace serves whichever it is (host only)."""
import pytest

from paper_2406_14066_amd import spec_verify as sv
from test_reject_plan_host import attn_args, reject_args


def plan(B, k, length, Hq, Hkv, d, with_reject=False):
    a = attn_args(B, k, length, Hq=Hq, Hkv=Hkv, d=d, dtype=sv.SPEC_F32, layout=sv.KV_TOKEN_MAJOR)
    p = sv.spec_verify_plan(a, reject_args(B, k, 1024) if with_reject else None)
    p["scalar"] = p["attn_blocks"] == p["max_chunks"] * a.Hq * a.T and p["chunk_tokens"] == 256
    return p


# few short requests on wide query groups: measured faster on the scalar kernel by 1.1 to 2.7 times
@pytest.mark.parametrize("B,k,length,Hq,Hkv,d", [(1, 4, 16, 64, 4, 128), (1, 4, 250, 64, 4, 128), (2, 4, 100, 64, 4, 128), (1, 8, 256, 16, 1, 128),
                                                 (4, 8, 128, 16, 1, 128), (1, 4, 16, 32, 8, 128), (2, 8, 32, 32, 8, 64)])
def test_few_short_requests_on_wide_groups_take_the_scalar_kernel(B, k, length, Hq, Hkv, d):
    p = plan(B, k, length, Hq, Hkv, d)
    assert p["scalar"] and p["launches"] == (2 if length > 256 else 1), p
    step = plan(B, k, length, Hq, Hkv, d, with_reject=True)
    assert not step["scalar"] and step["launches"] == 1, step     # beside the rejection half: one launch
    assert step["workspace_bytes"] >= p["workspace_bytes"]


@pytest.mark.parametrize("B,k,length,Hq,Hkv,d", [(8, 4, 1024, 32, 8, 128), (16, 4, 250, 64, 4, 128), (1, 4, 128, 32, 8, 128), (8, 4, 250, 64, 4, 128),
                                                 (1, 0, 128, 16, 8, 64), (48, 1, 16, 32, 8, 128), (64, 0, 16, 32, 16, 128), (2, 3, 256, 64, 4, 128)])
def test_others_take_the_matrix_instructions(B, k, length, Hq, Hkv, d):
    p = plan(B, k, length, Hq, Hkv, d)
    assert not p["scalar"] and p["launches"] == 1, p
