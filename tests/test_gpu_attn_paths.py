"""Every page walk of the attention kernels (wave groups that share their pages through LDS, K straight into
operand order, fp32) against the oracle: sizes at the edges of pages, tiles and rounds, and what the device
finds in lengths and block tables -- found once, left out or read as zeros, by whichever wavefront it falls to."""
import numpy as np
import pytest

import oracle
from paper_2406_14066_amd import spec_verify as sv
from paper_2406_14066_amd import workloads as W
from parity_utils import ATTN_TOL

pytestmark = pytest.mark.gpu

# dtype, query heads, KV heads, largest draft length, bf16: K straight into operand order, fp32: the scalar kernel; row tiles
# and wave groups of the matrix-instruction kernel
PATHS = [
    ("bf16", 8, 4, 4, 0, 1, 1), ("bf16", 8, 2, 7, 0, 2, 1), ("bf16", 8, 2, 7, 1, 2, 1), ("bf16", 16, 4, 8, 0, 3, 1),
    ("bf16", 16, 4, 8, 1, 3, 1), ("bf16", 16, 2, 6, 0, 2, 2), ("bf16", 16, 2, 6, 1, 2, 2), ("bf16", 16, 2, 8, 0, 3, 2),
    ("bf16", 16, 2, 8, 1, 3, 2), ("bf16", 32, 2, 6, 0, 2, 4), ("bf16", 16, 1, 8, 0, 3, 4),
    ("f32", 8, 4, 4, 0, 1, 1), ("f32", 8, 2, 7, 0, 2, 1), ("f32", 16, 2, 6, 0, 2, 2), ("f32", 16, 1, 8, 0, 3, 4), ("f32", 16, 1, 8, 1, 3, 4),
]
IDS = ["%s-%d-%d-k%d%s" % (p[0], p[1], p[2], p[3], ["-lds", "-direct", "-matrix", "-scalar"][p[4] + 2 * (p[0] == "f32")]) for p in PATHS]


def _setup(tuning, path, kv_len, k, **kw):
    from paper_2406_14066_amd.harness import DeviceStep
    dtype, Hq, Hkv, k_max, direct, tiles, groups = path
    tuning("SPEC_VERIFY_K_DIRECT" if dtype == "bf16" else "SPEC_VERIFY_F32_SCALAR", direct)
    # (the first request has the longest draft; others fill only some of the wave groups)
    w = W.make_workload("paths", B=len(kv_len), Hq=Hq, Hkv=Hkv, d=128, V=256, dtype=dtype, kv_len=list(kv_len),
                        k=[min(x, k_max) for x in k], draft_std=2.0, sigma=0.8, data_seed=Hq + k_max, philox_seed=9, **kw)
    ds = DeviceStep(w, kv_layout=sv.KV_TOKEN_MAJOR)
    plan = ds.plan()
    assert (plan["row_tiles"], plan["row_groups"]) == (tiles, groups), plan
    return w, ds


def _run(ds):
    """The attention alone; returns its output and what the device found."""
    import torch
    found = torch.zeros(1, dtype=torch.int64, device="cuda")
    ds.attn_args.error_count = found.data_ptr()
    ds.out.fill_(float("nan"))
    ds.run_attn()
    torch.cuda.synchronize()
    return ds.out.cpu().numpy(), int(found.item())


def _oracle(w):
    return oracle.verify_attn(w.q, w.k_pages, w.v_pages, w.block_table, w.kv_len, w.cu_q_len)


def _rows(w, b):
    return slice(int(w.cu_q_len[b]), int(w.cu_q_len[b + 1]))


@pytest.mark.parametrize("path", PATHS, ids=IDS)
@pytest.mark.parametrize("kv_len", [(9, 16, 17, 31, 64, 65, 127, 129, 255, 256), (257, 9, 300, 1000, 513, 64, 2049)], ids=["unsplit", "split"])
def test_lengths_at_page_and_round_edges(tuning, path, kv_len):
    print("case edges", path, kv_len, flush=True)
    w, ds = _setup(tuning, path, kv_len, [8, 0, 1, 8, 3, 5, 8, 0, 2, 8][: len(kv_len)])
    got, found = _run(ds)
    assert found == 0
    err = np.abs(got.astype(np.float64) - _oracle(w)).max()
    assert err <= ATTN_TOL[path[0]], err
    if path[0] == "bf16" and path[4] == 1:      # the same operands in the same order: the same bits as through LDS
        through_lds = list(path)
        through_lds[4] = 0
        _, ds0 = _setup(tuning, tuple(through_lds), kv_len, [8, 0, 1, 8, 3, 5, 8, 0, 2, 8][: len(kv_len)])
        np.testing.assert_array_equal(got, _run(ds0)[0])


@pytest.mark.parametrize("path", PATHS, ids=IDS)
def test_impossible_lengths_are_left_out_and_counted(tuning, path):
    import torch
    print("case bad lengths", path, flush=True)
    kv_len = (300, 45, 1000, 129, 64)
    for bad_b, bad_len in [(2, 5000), (1, 0), (0, -7)]:
        w, ds = _setup(tuning, path, kv_len, [8, 1, 4, 0, 2])
        dev_len = w.kv_len.copy()
        dev_len[bad_b] = bad_len
        ds.kv_len.copy_(torch.from_numpy(dev_len))
        got, found = _run(ds)
        assert found == 1, (bad_b, bad_len, found)
        assert np.isnan(got[_rows(w, bad_b)]).all()
        ok = np.ones(w.T, dtype=bool)
        ok[_rows(w, bad_b)] = False
        err = np.abs(got[ok].astype(np.float64) - _oracle(w)[ok]).max()
        assert err <= ATTN_TOL[path[0]], err


@pytest.mark.parametrize("path", PATHS, ids=IDS)
def test_bad_block_table_entries_read_as_zeros_and_are_counted_once(tuning, path):
    import torch
    print("case bad pages", path, flush=True)
    kv_len = (300, 45, 1000, 129, 64)
    bad = [(2, 7), (2, 30), (2, 62), (0, 18), (4, 0), (3, 8)]     # (request 2's and 0's last pages among them; request 3 fills one wave group)
    w, ds = _setup(tuning, path, kv_len, [8, 1, 4, 0, 2])
    table = w.block_table.copy()
    for i, (b, p) in enumerate(bad):
        table[b, p] = [w.num_blocks + 5, -3, 1 << 30][i % 3]
    ds.block_table.copy_(torch.from_numpy(table))
    got, found = _run(ds)
    assert found == len(bad), found
    assert np.isfinite(got).all()
    spare = [p for p in range(w.num_blocks) if p not in set(w.block_table.ravel().tolist())][: len(bad)]
    assert len(spare) == len(bad)
    for (b, i), p in zip(bad, spare):
        w.block_table[b, i] = p
        w.k_pages[p] = 0
        w.v_pages[p] = 0
    err = np.abs(got.astype(np.float64) - _oracle(w)).max()
    assert err <= ATTN_TOL[path[0]], err


# walks that take two pages at a time: a last page without a partner, one page, a page that a later chunk owns, short
# drafts that leave a tile or a group without rows, and values that are not finite past the end of a request
@pytest.mark.parametrize("kv_len", [(9, 16, 17, 33, 48, 49, 64, 65, 100, 129, 1000), (257, 9, 271, 1000, 513, 16, 2049)], ids=["unsplit", "split"])
@pytest.mark.parametrize("Hq,Hkv,d,k_max", [(8, 2, 64, 7), (16, 4, 64, 8), (32, 8, 64, 4), (16, 2, 64, 6), (16, 2, 64, 8), (32, 2, 64, 6), (16, 1, 64, 8),
                                            (16, 2, 128, 6), (32, 2, 128, 6)])
def test_pairs_of_pages(Hq, Hkv, d, k_max, kv_len):
    from paper_2406_14066_amd.harness import DeviceStep
    print("case pairs", Hq, Hkv, d, k_max, kv_len, flush=True)
    k = [min(x, k_max) for x in [8, 0, 1, 8, 3, 5, 8, 0, 2, 8, 8][: len(kv_len)]]
    w = W.make_workload("pairs", B=len(kv_len), Hq=Hq, Hkv=Hkv, d=d, V=256, dtype="bf16", kv_len=list(kv_len), k=k,
                        draft_std=2.0, sigma=0.8, data_seed=Hq + k_max + d, philox_seed=9)
    inf = np.uint16(0x7F80) if w.v_pages.dtype == np.uint16 else np.inf
    for b, n in enumerate(kv_len):
        if n % 16:
            w.v_pages[w.block_table[b, n // 16], :, n % 16:] = inf
            w.k_pages[w.block_table[b, n // 16], :, n % 16:] = inf
    ds = DeviceStep(w, kv_layout=sv.KV_TOKEN_MAJOR)
    got, found = _run(ds)
    assert found == 0
    err = np.abs(got.astype(np.float64) - _oracle(w)).max()
    assert err <= ATTN_TOL["bf16"], err


# chunks sized from all lengths: the grid lists the chunks that exist; lengths that do not fit are left out and counted once,
# and a workspace that holds the partial results of the longest request's split only serves with that split
@pytest.mark.parametrize("dtype,Hq,Hkv,k,kv_len,chunks", [
    ("bf16", 8, 8, 3, (5000, 513, 16, 9, 2000, 3100, 700, 40), 8), ("f32", 16, 8, 8, (1000, 9, 500, 200), 6), ("f32", 32, 8, 4, (500,), 4),
    ("bf16", 16, 16, 2, (4000, 600, 64, 6000), 8)])
def test_chunks_sized_from_all_lengths(dtype, Hq, Hkv, k, kv_len, chunks):
    from paper_2406_14066_amd.harness import DeviceStep
    print("case spread", dtype, Hq, Hkv, k, kv_len, flush=True)
    w = W.make_workload("spread", B=len(kv_len), Hq=Hq, Hkv=Hkv, d=128, V=256, dtype=dtype, kv_len=list(kv_len),
                        k=[min(k, n - 1) for n in kv_len], draft_std=2.0, sigma=0.8, data_seed=Hq + k, philox_seed=9)
    ds = DeviceStep(w, kv_layout=sv.KV_TOKEN_MAJOR)
    plan = sv.spec_verify_plan(ds.attn_args, None)
    need = sum((n + plan["chunk_tokens"] - 1) // plan["chunk_tokens"] for n in kv_len) * Hkv
    assert plan["max_chunks"] == chunks and need <= 256, (plan, need)
    ref = _oracle(w)
    got, found = _run(ds)
    assert found == 0
    assert np.abs(got.astype(np.float64) - ref).max() <= ATTN_TOL[dtype]
    # the split of the longest request alone, which is what a bucket of that length gets
    import ctypes
    bucket = type(ds.attn_args)()
    ctypes.memmove(ctypes.byref(bucket), ctypes.byref(ds.attn_args), ctypes.sizeof(bucket))
    bucket.max_kv_len = max(kv_len)
    small = sv.spec_verify_workspace_bytes(bucket, None)
    whole = ds.workspace
    if small < sv.spec_verify_workspace_bytes(ds.attn_args, None):
        ds.workspace = whole[:small]
        got, found = _run(ds)
        assert found == 0
        assert np.abs(got.astype(np.float64) - ref).max() <= ATTN_TOL[dtype]
        ds.workspace = whole
    if len(kv_len) == 1:
        return
    assert plan["attn_blocks"] == need, plan
    # a length beyond the plan and one below its own query rows
    good = ds.kv_len.clone()
    bad = {0: plan["chunk_tokens"] * plan["max_chunks"] + 1, 2: 0}
    for b, n in bad.items():
        ds.kv_len[b] = n
    got, found = _run(ds)
    ds.kv_len.copy_(good)
    assert found == len(bad)
    for b in range(w.B):
        rows = got[_rows(w, b)]
        if b in bad:
            assert np.isnan(rows).all()
        else:
            assert np.abs(rows.astype(np.float64) - ref[_rows(w, b)]).max() <= ATTN_TOL[dtype]


# requests of two to four chunks, whose merge takes four rows of four chunks per half wavefront and pass: 17 to 64 rows
@pytest.mark.parametrize("dtype,Hq,Hkv,k_max", [("bf16", 16, 2, 6), ("bf16", 16, 2, 7), ("f32", 8, 2, 7), ("f32", 9, 1, 1), ("f32", 16, 2, 6), ("f32", 32, 2, 7)])
def test_merge_of_few_chunks(tuning, dtype, Hq, Hkv, k_max):
    from paper_2406_14066_amd.harness import DeviceStep
    print("case few chunks", dtype, Hq, Hkv, k_max, flush=True)
    tuning("SPEC_VERIFY_F32_SCALAR", 0)
    kv_len = (1000, 257, 513, 40, 769)
    w = W.make_workload("merge", B=len(kv_len), Hq=Hq, Hkv=Hkv, d=128, V=256, dtype=dtype, kv_len=list(kv_len),
                        k=[min(x, k_max) for x in (8, 0, 8, 3, 2)], draft_std=2.0, sigma=0.8, data_seed=Hq + k_max, philox_seed=9)
    ds = DeviceStep(w, kv_layout=sv.KV_TOKEN_MAJOR)
    assert ds.plan()["max_chunks"] == 4, ds.plan()
    got, found = _run(ds)
    assert found == 0
    assert np.abs(got.astype(np.float64) - _oracle(w)).max() <= ATTN_TOL[dtype]


# the listed chunks are the host lengths': a request that has grown or shrunk on the device is served with them, in longer ones if
# they are too few, up to 64 pages per wavefront; one that does not fit those is left out and counted once
@pytest.mark.parametrize("dtype,Hq,Hkv,k,groups", [("bf16", 16, 16, 2, 1), ("f32", 16, 8, 2, 1), ("bf16", 64, 8, 7, 2), ("f32", 64, 8, 7, 2)])
def test_lengths_that_outgrow_their_listed_chunks(dtype, Hq, Hkv, k, groups):
    from paper_2406_14066_amd.harness import DeviceStep
    print("case outgrown", dtype, Hq, Hkv, k, flush=True)
    kv_len = (4000, 600, 64, 6000) + (100,) * (4 if groups == 2 else 0)
    w = W.make_workload("outgrown", B=len(kv_len), Hq=Hq, Hkv=Hkv, d=128, V=256, dtype=dtype, kv_len=list(kv_len), k=[k] * len(kv_len), draft_std=2.0, sigma=0.8,
                        data_seed=Hq, philox_seed=9)
    w.block_table = np.concatenate([w.block_table, w.block_table], axis=1)   # room for the longer lengths (any pages will do)
    ds = DeviceStep(w, kv_layout=sv.KV_TOKEN_MAJOR)
    plan = sv.spec_verify_plan(ds.attn_args, None)
    C = plan["chunk_tokens"]
    chunks = [(n + C - 1) // C for n in kv_len]
    assert plan["attn_blocks"] == Hkv * sum(chunks) < Hkv * len(kv_len) * plan["max_chunks"] and plan["row_groups"] == groups, plan
    most, bound = 4096 // groups, C * plan["max_chunks"]    # tokens of a chunk, of a request
    for b in (0, 1, 2):
        w.block_table[b] = np.resize(w.block_table[3, : 6000 // 16], w.block_table.shape[1])
    ds.block_table.copy_(ds.block_table.new_tensor(w.block_table))
    one, two = min(chunks[2] * most, bound), min(chunks[1] * most, bound)    # (what a request of one chunk and one of some can grow to)
    cases = [([chunks[0] * C, 500, 40, 3000], ()), ([chunks[0] * C + 1, 500, 64, 6000], ()), ([4000, chunks[1] * C + 16, C + 1, 6000], ()),
             ([4000, two, one, 17], ())]
    if chunks[2] * most < bound:
        cases.append(([4000, 600, chunks[2] * most + 1, 6000], (2,)))
    for lens, out in cases:
        w.kv_len = np.asarray(tuple(lens) + kv_len[4:], dtype=np.int32)
        ds.kv_len.copy_(ds.kv_len.new_tensor(w.kv_len))
        got, found = _run(ds)
        assert found == len(out), (lens, found)
        ref = _oracle(w)
        for b in range(w.B):
            rows = got[_rows(w, b)]
            if b in out:
                assert np.isnan(rows).all()
            else:
                assert np.abs(rows.astype(np.float64) - ref[_rows(w, b)]).max() <= ATTN_TOL[dtype], (lens, b)
