"""Performance cases of the speculative-verification library: what a serving engine has it do,
over the range of batch sizes, context lengths, draft lengths, head shapes, vocabularies, page
layouts, data types and acceptance modes that the library is meant for.

A case is a dict of plain values.  `path` names the entry point:

  step    spec_verify_step: lookahead attention and rejection sampling in one call
  attn    spec_verify_attn: the attention alone (an engine calls it once per layer)
  reject  spec_reject_sample: the rejection sampling alone (once per step)
  append  spec_kv_append: the step's K/V rows into the paged cache (once per layer)
  repack  spec_kv_repack_mfma: a token-major page pool into the tiled page layout

Context lengths and draft lengths are derived from the case alone (`lmin`..`lmax`, `k` or, with
`ragged_k`, 1..k per request), so that a case has one amount of work; everything else (queries,
cache contents, block tables, logits, draft tokens) is drawn from the seed.
"""
import math
import random

import torch

from paper_2406_14066_amd import spec_verify as sv

PAGE = 16
MODES = {"sample": sv.ACCEPT_SAMPLE, "greedy": sv.ACCEPT_GREEDY, "point": sv.ACCEPT_POINT_DRAFT}


def listed():
    step = dict(path="step", ragged_k=False, dtype="bf16", d=128, layout="tiles", mode="sample", bucket=False)
    attn = dict(path="attn", ragged_k=False, dtype="bf16", d=128, layout="tiles", bucket=False)
    return [
        # The smallest call there is: the fp32 toy model (8 heads of 64, 128 tokens, a vocabulary of
        # 1024), as one checks an integration with.  Launches and latencies only.
        dict(step, name="step_tiny_f32", B=1, k=4, lmin=128, lmax=128, Hq=8, Hkv=8, d=64, dtype="f32",
             layout="tokens", V=1024),
        # One interactive user of a 70B-shaped model, under a length bucket as a captured decode loop
        # uses it: the latency of a step that nothing else hides.
        dict(step, name="step_one_request", B=1, k=4, lmin=687, lmax=687, Hq=64, Hkv=8, V=32000, bucket=True),
        # A small batch of a Llama-2-7B-shaped model (no grouped heads) at 2048 tokens, k = 4.
        dict(step, name="step_7b_batch8", B=8, k=4, lmin=2048, lmax=2048, Hq=32, Hkv=32, V=32000),
        # The full batch of a 70B-shaped model (64/8 heads), ragged contexts of the length of chat and
        # summarisation traces: the busy server.
        dict(step, name="step_70b_batch256", B=256, k=2, lmin=256, lmax=1024, Hq=64, Hkv=8, V=32000),
        # The same model at a high acceptance rate (k = 7: 64 fused query rows per KV head) on an
        # engine that keeps its own token-major pages.
        dict(step, name="step_70b_k7_token_pages", B=96, k=7, lmin=256, lmax=1024, Hq=64, Hkv=8, V=32000,
             layout="tokens"),
        # A few long documents with draft lengths chosen per request, large vocabulary.
        dict(step, name="step_long_context", B=4, k=8, ragged_k=True, lmin=6000, lmax=32768, Hq=32, Hkv=8,
             V=128256),
        # One layer of a small grouped-head model (head dim 64) on token-major pages.
        dict(attn, name="attn_d64_token_pages", B=64, k=3, lmin=200, lmax=1900, Hq=32, Hkv=8, d=64, layout="tokens"),
        # One layer of a grouped-head model run in fp32, as an engine does to check a model's numerics.
        dict(attn, name="attn_f32", B=8, k=4, lmin=256, lmax=1024, Hq=32, Hkv=8, dtype="f32", layout="tokens"),
        # Acceptance for a batch with per-request draft lengths and a large vocabulary.
        dict(path="reject", name="reject_sample_128k", B=48, k=6, ragged_k=True, V=128256, mode="sample"),
        # Greedy acceptance (temperature 0) for a full batch.
        dict(path="reject", name="reject_greedy_32k", B=256, k=3, ragged_k=False, V=32000, mode="greedy"),
        # The K/V rows of a full batch's step enter one layer's cache.
        dict(path="append", name="append_batch256", B=256, k=4, lmin=256, lmax=1024, Hkv=8, d=128, dtype="bf16",
             layout="tiles"),
        # A cache filled by a prefill that writes token-major pages is taken over.
        dict(path="repack", name="repack_pool", pages=4096, Hkv=8, d=128),
    ]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    path = rng.choice(["step", "step", "step", "attn", "attn", "reject", "reject", "append", "repack"])
    heads = rng.choice([(32, 32, 128), (32, 8, 128), (64, 8, 128), (64, 4, 128), (16, 16, 64), (32, 8, 64)])
    vocab = rng.choice([32000, 128256, 4 * _log_int(rng, 256, 38016)])
    if path == "repack":
        return dict(path=path, pages=_log_int(rng, 16, 8192), Hkv=rng.choice([4, 8, 16]), d=rng.choice([64, 128]))
    k = rng.randint(0, 8)
    ragged_k = k > 1 and rng.random() < 0.4
    if path == "reject":
        rows = 200e6 / (vocab * 4)      # logit rows that fit the bytes of the larger listed cases
        B = _log_int(rng, 1, max(1, min(256, int(rows / (2 * k + 1)))))
        return dict(path=path, B=B, k=k, ragged_k=ragged_k, V=vocab, mode=rng.choice(["sample", "sample", "greedy", "point"]))
    Hq, Hkv, d = heads
    B = _log_int(rng, 1, 256)
    f32 = path != "append" and rng.random() < 0.2
    layout = "tokens" if f32 else rng.choice(["tiles", "tokens"])
    # tokens per request whose K and V, and whose arithmetic, fit the larger listed cases
    longest = min(500e6 / (B * Hkv * d * 4), 16e9 / (4 * B * (k + 1) * Hq * d))
    if f32:
        longest = min(longest, 1.0e6 * 128 * 8 / (B * (k + 1) * Hq * d))
    mean = _log_int(rng, 32, int(max(40, min(32768, longest))))
    spread = rng.choice([0.0, 0.3, 0.9])
    lmin, lmax = max(k + 1, int(mean * (1 - spread))), max(k + 1, int(mean * (1 + spread)))
    if path == "append":
        return dict(path=path, B=B, k=k, lmin=lmin, lmax=lmax, Hkv=Hkv, d=d, dtype=rng.choice(["bf16", "bf16", "f32"]),
                    layout="tokens") if layout == "tokens" else \
            dict(path=path, B=B, k=k, lmin=lmin, lmax=lmax, Hkv=Hkv, d=d, dtype="bf16", layout="tiles")
    case = dict(path=path, B=B, k=k, ragged_k=ragged_k, lmin=lmin, lmax=lmax, Hq=Hq, Hkv=Hkv, d=d,
                dtype="f32" if f32 else "bf16", layout=layout, bucket=rng.random() < 0.3)
    if path == "step":
        while B * (2 * k + 1) * vocab * 4 > 250e6 and vocab > 1024:
            vocab = vocab // 8 * 4
        case.update(V=vocab, mode=rng.choice(["sample", "sample", "greedy", "point"]))
    return case


# --------------------------------------------------------------------------- inputs
def _q_lens(case):
    rng = random.Random("q %d %d" % (case["B"], case["k"]))
    if case.get("ragged_k"):
        return [rng.randint(1, case["k"]) + 1 for _ in range(case["B"])]
    return [case["k"] + 1] * case["B"]


def _kv_lens(case):
    rng = random.Random("kv %d %d %d" % (case["B"], case["lmin"], case["lmax"]))
    return [max(rng.randint(case["lmin"], case["lmax"]), q) for q in _q_lens(case)]


def _prefix(lens):
    out = [0]
    for n in lens:
        out.append(out[-1] + n)
    return out


def _gen(seed, salt):
    g = torch.Generator(device="cuda")
    g.manual_seed((int(seed) * 1000003 + salt) & 0x7FFFFFFFFFFF)
    return g


def _i32(values):
    return torch.tensor(values, dtype=torch.int32)


def _normal(shape, dtype, g):
    return torch.randn(shape, dtype=torch.float32, device="cuda", generator=g).to(dtype)


def _dtype(case):
    return torch.float32 if case["dtype"] == "f32" else torch.bfloat16


def _table(case, g):
    """A shuffled block table over a pool with a quarter of its pages spare."""
    pages = [(n + PAGE - 1) // PAGE for n in _kv_lens(case)]
    need = sum(pages)
    blocks = need + (need + 3) // 4
    order = torch.randperm(blocks, device="cuda", generator=g)[:need].to(torch.int32)
    table = torch.zeros((case["B"], max(pages)), dtype=torch.int32, device="cuda")
    at = torch.arange(max(pages), device="cuda")[None, :] < torch.tensor(pages, device="cuda")[:, None]
    table[at] = order
    return table, blocks


def _attn_inputs(case, seed):
    """Queries, token-major page pools and the block table."""
    g = _gen(seed, 1)
    T, d = sum(_q_lens(case)), case["d"]
    table, blocks = _table(case, g)
    q = _normal((T, case["Hq"], d), _dtype(case), g)
    k = _normal((blocks, case["Hkv"], PAGE, d), _dtype(case), g)
    v = _normal((blocks, case["Hkv"], PAGE, d), _dtype(case), g)
    return q, k, v, table


def _logits(case, seed):
    """Draft rows ~ N(0, 3^2), target row = draft row + N(0, 0.77^2) (an acceptance rate of about 0.7),
    one more target row per request, draft tokens drawn from the softmax of their row (for the greedy
    mode: its arg-max, which is what a greedy proposer gives)."""
    g = _gen(seed, 2)
    q_lens, V = _q_lens(case), case["V"]
    T, B = sum(q_lens), case["B"]
    draft = torch.randn((T, V), device="cuda", generator=g) * 3.0
    target = draft + torch.randn((T, V), device="cuda", generator=g) * 0.77
    keep = torch.ones(T, dtype=torch.bool, device="cuda")
    keep[torch.tensor(_prefix(q_lens)[1:], device="cuda") - 1] = False
    draft = draft[keep].contiguous()
    if T == B:
        return target, None, None
    if case["mode"] == "greedy":
        tokens = draft.argmax(1)
    else:
        noise = torch.empty_like(draft).exponential_(generator=g)
        tokens = (draft - noise.log()).argmax(1)
    return target, draft, tokens.to(torch.int32)


class _State:
    pass


def _attn_state(s, case, seed):
    q, k, v, table = _attn_inputs(case, seed)
    layout = sv.KV_TOKEN_MAJOR
    if case["layout"] == "tiles":
        kt, vt = torch.empty_like(k), torch.empty_like(v)
        sv.spec_kv_repack_mfma(k, v, kt, vt)
        k, v, layout = kt, vt, sv.KV_MFMA
    kv_lens = _kv_lens(case)
    s.out = torch.zeros((q.shape[0], case["Hq"], case["d"]), device="cuda")
    bound = (max(kv_lens) + 255) // 256 * 256 if case["bucket"] else 0
    if bound:   # a bucket's table has room for its longest request
        table = torch.nn.functional.pad(table, (0, bound // PAGE - table.shape[1])).contiguous()
    s.kv_len = _i32(kv_lens).cuda()
    s.attn, s.keep_attn = sv.make_attn_args(
        q, k, v, table, s.kv_len, s.cu, s.out, kv_lens, s.host_cu, Hkv=case["Hkv"], kv_layout=layout, max_kv_len=bound)


def _reject_state(s, case, seed):
    B = case["B"]
    target, draft, tokens = _logits(case, seed)
    T = target.shape[0]
    s.outputs = dict(
        accepted_len=torch.zeros(B, dtype=torch.int32, device="cuda"),
        next_token=torch.zeros(B, dtype=torch.int32, device="cuda"),
        out_tokens=torch.zeros((B, sv.K_MAX + 1), dtype=torch.int32, device="cuda"),
        counters=torch.zeros(sv.NUM_COUNTERS, dtype=torch.int64, device="cuda"))
    u_ratio = None
    if case["mode"] != "greedy" and T > B:
        u_ratio = s.outputs["u_ratio"] = torch.zeros((T - B, 2), dtype=torch.float64, device="cuda")
    more = {}
    if case["path"] == "step":      # a decode loop takes the new cache lengths from the step
        s.outputs["new_kv_len"] = torch.zeros(B, dtype=torch.int32, device="cuda")
        more = dict(kv_len=s.kv_len, new_kv_len=s.outputs["new_kv_len"])
    s.reject, s.keep_reject = sv.make_reject_args(
        target, draft, tokens, s.cu, s.host_cu, s.outputs["accepted_len"], s.outputs["next_token"],
        s.outputs["counters"], philox_seed=int(seed), philox_step=7, out_tokens=s.outputs["out_tokens"],
        debug_u_ratio=u_ratio, accept_mode=MODES[case["mode"]], **more)


def prepare(case, seed):
    s = _State()
    s.path = case["path"]
    if s.path == "repack":
        g = _gen(seed, 3)
        shape = (case["pages"], case["Hkv"], PAGE, case["d"])
        s.src_k, s.src_v = _normal(shape, torch.bfloat16, g), _normal(shape, torch.bfloat16, g)
        s.dst_k, s.dst_v = torch.empty_like(s.src_k), torch.empty_like(s.src_v)
        return s
    s.host_cu = _prefix(_q_lens(case))
    s.cu = _i32(s.host_cu).cuda()
    if s.path == "append":
        g = _gen(seed, 4)
        table, blocks = _table(case, g)
        kv_lens = _kv_lens(case)
        pool = (blocks, case["Hkv"], PAGE, case["d"])
        rows = (s.host_cu[-1], case["Hkv"], case["d"])
        s.k_cache, s.v_cache = _normal(pool, _dtype(case), g), _normal(pool, _dtype(case), g)
        new_k, new_v = _normal(rows, _dtype(case), g), _normal(rows, _dtype(case), g)
        s.append, s.keep = sv.make_kv_append_args(
            new_k, new_v, s.k_cache, s.v_cache, table, _i32(kv_lens).cuda(), s.cu, kv_lens, s.host_cu,
            kv_layout=sv.KV_MFMA if case["layout"] == "tiles" else sv.KV_TOKEN_MAJOR)
        return s
    s.attn = s.reject = None
    if s.path in ("step", "attn"):
        _attn_state(s, case, seed)
    if s.path in ("step", "reject"):
        _reject_state(s, case, seed)
    s.workspace = sv.alloc_workspace(sv.spec_verify_workspace_bytes(s.attn, s.reject))
    return s


def run(s):
    if s.path == "step":
        sv.spec_verify_step(s.attn, s.reject, s.workspace)
        return dict(s.outputs, out=s.out)
    if s.path == "attn":
        sv.spec_verify_attn(s.attn, s.workspace)
        return dict(out=s.out)
    if s.path == "reject":
        sv.spec_reject_sample(s.reject, s.workspace)
        return s.outputs
    if s.path == "append":
        sv.spec_kv_append_args(s.append)
        return dict(k_cache=s.k_cache, v_cache=s.v_cache)
    sv.spec_kv_repack_mfma(s.src_k, s.src_v, s.dst_k, s.dst_v)
    return dict(k=s.dst_k, v=s.dst_v)


# --------------------------------------------------------------------------- work, tolerance
def work(case):
    if case["path"] == "repack":
        return {"bytes": 4 * case["pages"] * case["Hkv"] * PAGE * case["d"] * 2, "flops": 0}
    q_lens = _q_lens(case)
    T, B = sum(q_lens), case["B"]
    nbytes = flops = 0
    if case["path"] == "append":    # new rows read, and written to the cache
        return {"bytes": 4 * T * case["Hkv"] * case["d"] * (4 if case["dtype"] == "f32" else 2) + 12 * B, "flops": 0}
    if case["path"] in ("step", "attn"):
        esz = 4 if case["dtype"] == "f32" else 2
        lens, d = _kv_lens(case), case["d"]
        nbytes += sum(lens) * case["Hkv"] * d * 2 * esz                 # K and V once
        nbytes += T * case["Hq"] * d * (esz + 4)                        # queries in, fp32 output
        nbytes += 4 * sum((n + PAGE - 1) // PAGE for n in lens)         # block table
        flops += sum(4 * n * q * case["Hq"] * d for n, q in zip(lens, q_lens))
    if case["path"] in ("step", "reject"):
        rows = 2 * T - B if case["mode"] == "sample" else T             # every logit row once
        nbytes += rows * case["V"] * 4
        flops += rows * case["V"] * (2 if case["mode"] == "greedy" else 4)
    return {"bytes": nbytes, "flops": flops}


def tolerance(case):
    if case["path"] in ("append", "repack") or (case["path"] == "reject" and case["mode"] == "greedy"):
        return "exact"
    # `differ`: a decision within rounding of its threshold may fall the other way (one in a large batch).
    if case["path"] == "reject" or case["dtype"] == "f32":
        # p/q of the draft tokens from fp32 exponentials and fp64 sums (7e-8 off the 64-bit result); fp32
        # attention (4e-7 off)
        return {"rel": 2e-6, "max": 8e-5, "differ": 0.005}
    # bf16 cache and queries, softmax weights as bf16 high + low parts, fp32 accumulation and output
    # (2.4e-6 off the 64-bit result)
    return {"rel": 1e-5, "max": 4e-4, "differ": 0.005}


# --------------------------------------------------------------------------- 64-bit reference
def _exact_attention(case, seed):
    q, k, v, table = _attn_inputs(case, seed)
    cu, lens = _prefix(_q_lens(case)), _kv_lens(case)
    Hq, Hkv, d = case["Hq"], case["Hkv"], case["d"]
    out = torch.empty((cu[-1], Hq, d), dtype=torch.float64, device="cuda")
    for b, n in enumerate(lens):
        pages = table[b, : (n + PAGE - 1) // PAGE].long()
        keys = k[pages].transpose(0, 1).reshape(Hkv, -1, d)[:, :n].double()
        values = v[pages].transpose(0, 1).reshape(Hkv, -1, d)[:, :n].double()
        m = cu[b + 1] - cu[b]
        rows = q[cu[b]:cu[b + 1]].double().reshape(m, Hkv, Hq // Hkv, d).permute(1, 0, 2, 3).reshape(Hkv, -1, d)
        s = torch.matmul(rows, keys.transpose(1, 2).contiguous()) / math.sqrt(d)
        last = n - m + torch.arange(m, device="cuda").repeat_interleave(Hq // Hkv)
        s.masked_fill_(torch.arange(n, device="cuda")[None, None, :] > last[None, :, None], -math.inf)
        o = torch.matmul(torch.softmax(s, -1), values)
        out[cu[b]:cu[b + 1]] = o.reshape(Hkv, m, Hq // Hkv, d).permute(1, 0, 2, 3).reshape(m, Hq, d)
    return out


def _philox_word0(index, b, step, key):
    """First word of Philox4x32-10 with counter (index, b, step, stream 0), as Python integers."""
    c, k0, k1 = [index, b, step & 0xFFFFFFFF, ((step >> 32) & 0xFFFFFF) << 8], key & 0xFFFFFFFF, (key >> 32) & 0xFFFFFFFF
    for _ in range(10):
        pa, pb = 0xD2511F53 * c[0], 0xCD9E8D57 * c[2]
        c = [(pb >> 32) ^ c[1] ^ k0, pb & 0xFFFFFFFF, (pa >> 32) ^ c[3] ^ k1, pa & 0xFFFFFFFF]
        k0, k1 = (k0 + 0x9E3779B9) & 0xFFFFFFFF, (k1 + 0xBB67AE85) & 0xFFFFFFFF
    return c[0]


def _exact_u_ratio(case, seed):
    """u and p/q of every accept test up to a request's first rejection, NaN after it."""
    target, draft, tokens = _logits(case, seed)
    cu, B = _prefix(_q_lens(case)), case["B"]
    out = torch.full((cu[-1] - B, 2), math.nan, dtype=torch.float64)
    log_p, log_q = [], []
    at = [(b, i) for b in range(B) for i in range(cu[b + 1] - cu[b] - 1)]
    for r, (b, i) in enumerate(at):
        x = tokens[r].long()
        row = target[cu[b] + i].double()
        log_p.append(row[x] - torch.logsumexp(row, 0))
        if case["mode"] == "sample":
            row = draft[r].double()
            log_q.append(row[x] - torch.logsumexp(row, 0))
        else:
            log_q.append(torch.zeros((), dtype=torch.float64, device="cuda"))
    ratio = torch.exp(torch.stack(log_p) - torch.stack(log_q)).cpu()
    over = set()
    for r, (b, i) in enumerate(at):
        if b in over:
            continue
        u = (_philox_word0(i, b, 7, int(seed)) >> 8) / 16777216.0
        out[r, 0], out[r, 1] = u, ratio[r]
        if not u < float(ratio[r]):
            over.add(b)
    return out.cuda()


def exact(case, seed):
    path = case["path"]
    if path in ("append", "repack"):
        return None     # bytes moved: compared as they are
    answer = {}
    if path in ("step", "reject"):
        answer = dict(accepted_len=None, next_token=None, out_tokens=None, counters=None)
        if path == "step":
            answer["new_kv_len"] = None
        if case["mode"] != "greedy" and sum(_q_lens(case)) > case["B"]:
            answer["u_ratio"] = _exact_u_ratio(case, seed)
    if path in ("step", "attn"):
        answer["out"] = _exact_attention(case, seed)
    return answer if any(v is not None for v in answer.values()) else None
