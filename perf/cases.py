"""Performance cases of the sampler: what a serving loop calls, over the sizes it meets.

A case is a plain dict.  Its fields:

  op      entry point of ``paper_2607_20475_amd.binding``: sample, sample_full, sample_gumbel,
          logprobs, topk, verify, verify_tree or process
  dtype   logits type, bf16 or f32
  B, V    requests, vocabulary (rows are contiguous, so an odd V leaves rows unaligned)
  L       draft length (verification), 0 elsewhere
  k_max   candidate bound (entries per row for logprobs and topk)
  k_out   entries of the kept list that sample returns, 0 for none
  k       ``all`` (top-k drawn from 1..k_max per request), ``off`` (no top-k cut) or ``fix`` (k = k_max)
  hist    ids of each request's penalty history; with it go 16 logit biases per request; 0 for neither
  grammar whether an allow bitmask of 5 % of the ids applies

Logits are concentrated next-token distributions: N(0, 2) with a few ids raised by U(8, 16).
Tokens, log-probabilities, lists, accepted counts and materialised rows are returned.  The
flags are not: beside two bits that follow from the inputs they hold one that names the
internal path a row took, which is no result.
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2607_20475_amd import binding as ssb

PENALTIES = ssb.REP | ssb.FREQ | ssb.PRES | ssb.BIAS
NBIAS = 16
KQ = 64       # entries of a sparse draft list
EXTRA_ROWS = 4  # target rows of a draft tree beside the verified path


def listed():
    def case(name, op, dtype, B, V, L=0, k_max=1024, k_out=0, k="all", hist=512, grammar=False):
        return dict(name=name, op=op, dtype=dtype, B=B, V=V, L=L, k_max=k_max, k_out=k_out, k=k, hist=hist,
                    grammar=grammar)

    return [
        # a few interactive users, small vocabulary, float32 logits, mixed temperatures: latency
        case("sample_b4_f32", "sample", "f32", 4, 32768, k_max=64, k="fix", hist=0),
        # a decode step of a serving batch: greedy and stochastic requests, penalties, biases
        case("sample_b64_bf16", "sample", "bf16", 64, 131072),
        # the same with grammar-constrained requests
        case("sample_grammar_b128_bf16", "sample", "bf16", 128, 131072, grammar=True),
        # a large vocabulary that is not padded: odd row length, rows at odd addresses
        case("sample_odd_b48_bf16", "sample", "bf16", 48, 200003),
        # a draft model's step: the kept list with its probabilities goes on to verification
        case("sample_list_b64_bf16", "sample", "bf16", 64, 131072, k_max=64, k_out=64, k="fix", hist=0),
        # nucleus sampling over the whole row: top-p / min-p, no top-k cut
        case("sample_full_b64_bf16", "sample_full", "bf16", 64, 131072, k="off"),
        # the draw by noise that the caller made
        case("sample_gumbel_b64_bf16", "sample_gumbel", "bf16", 64, 131072),
        # log-probabilities of the leading tokens, as an API returns them
        case("logprobs_b64_bf16", "logprobs", "bf16", 64, 131072, k_max=20),
        # top-k alone, large batch and vocabulary, float32, k from 1 to 4096; the largest call
        case("topk_b256_f32", "topk", "f32", 256, 262144, k_max=4096, hist=0),
        # verification of four drafts a request against the draft model's dense probabilities
        case("verify_b64_l4_bf16", "verify", "bf16", 64, 131072, L=4),
        # verification of a path in a draft tree against sparse draft lists
        case("verify_tree_b32_l6_bf16", "verify_tree", "bf16", 32, 131072, L=6),
        # the whole processed row and its final distribution, for callers that go on from there
        case("process_b32_bf16", "process", "bf16", 32, 131072),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    op = rng.choice(["sample", "sample", "sample", "sample_full", "sample_gumbel", "logprobs", "topk", "verify",
                     "verify_tree", "process"])
    dtype = rng.choice(["bf16", "bf16", "f32"])
    V = _log_int(rng, 32000, 262144)
    V = rng.choice([V, V | 1, (V + 63) // 64 * 64, (V + 63) // 64 * 64])
    verify = op in ("verify", "verify_tree")
    B = _log_int(rng, 1, 64 if verify or op == "process" else 256)
    L = rng.randint(1, 8) if verify else 0
    while B * (L + 1) > 384 or (op == "sample_gumbel" and B > 128) or B * (L + 1) * V > 48e6:
        B = max(1, B // 2)
    k_max = rng.choice([5, 20, 64]) if op == "logprobs" else rng.choice([64, 256, 1024, 1024, 4096])
    k = "off" if op == "sample_full" else rng.choice(["all", "all", "all", "fix"])
    k_out = rng.choice([0, 0, 64]) if op == "sample" else 0
    hist = 0 if op == "topk" else rng.choice([0, _log_int(rng, 16, 1024), _log_int(rng, 16, 1024)])
    return dict(op=op, dtype=dtype, B=B, V=V, L=L, k_max=k_max, k_out=k_out, k=k, hist=hist,
                grammar=op != "topk" and rng.random() < 0.25)


# ---------------------------------------------------------------------------
# Inputs (all on the GPU, from the seed alone)
# ---------------------------------------------------------------------------
def _spread(g, rows, n, V):
    """n distinct ids per row, one from each of n equal stretches of the vocabulary."""
    w = V // n
    at = torch.randint(0, w, (rows, n), generator=g, device="cuda")
    return at + torch.arange(n, device="cuda") * w


def _logits(g, rows, V, heads):
    x = torch.empty(rows, V, device="cuda").normal_(0.0, 2.0, generator=g)
    ids = _spread(g, rows, heads, V)
    x.scatter_add_(1, ids, torch.empty(rows, heads, device="cuda").uniform_(8.0, 16.0, generator=g))
    return x


def _exponential(g, *shape):
    return torch.empty(*shape, device="cuda").exponential_(1.0, generator=g).clamp_min_(1e-30)


def _inputs(case, seed):
    """What the call reads, as a dict of tensors (also what ``exact`` starts from)."""
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed) * 2654435761 % (1 << 62) + 7)
    op, B, V, L, k_max = case["op"], case["B"], case["V"], case["L"], case["k_max"]
    verify = op in ("verify", "verify_tree")
    rows = B * (L + 1) if verify else B
    uni = lambda lo, hi: torch.empty(B, device="cuda").uniform_(lo, hi, generator=g)  # noqa: E731
    d = {}
    x = _logits(g, rows, V, 32 if op == "topk" else 16)
    if op == "topk":  # every other row is flat, as an untrained or high-temperature head gives
        x[1::2] = torch.empty(B // 2, V, device="cuda").uniform_(-1.0, 1.0, generator=g)
    x = x.to(torch.bfloat16 if case["dtype"] == "bf16" else torch.float32)
    odd = (torch.arange(B, device="cuda") % 2 == 1)
    d["top_k"] = torch.randint(1, k_max + 1, (B,), generator=g, device="cuda").to(torch.int32) if case["k"] == "all" \
        else torch.full((B,), k_max if case["k"] == "fix" else 0, dtype=torch.int32, device="cuda")
    if op == "topk":  # greedy, usual and very long lists side by side
        d["top_k"] = torch.tensor([1, 50, 1024, 4096], dtype=torch.int32, device="cuda").clamp_max(k_max)[
            torch.randint(0, 4, (B,), generator=g, device="cuda")]
        d["x"] = x
        return d
    trunc = ssb.TEMP | ssb.TOPP | ssb.MINP | (ssb.TOPK if case["k"] != "off" else 0)
    if op == "logprobs":
        mode = torch.full((B,), ssb.TEMP | ssb.LOGPROBS, dtype=torch.int32, device="cuda")
    elif case["k"] == "fix":  # every request stochastic but those at temperature zero
        mode = torch.full((B,), trunc, dtype=torch.int32, device="cuda")
    else:
        mode = torch.where(odd, trunc, ssb.GREEDY).to(torch.int32)
    d["temperature"] = uni(0.3, 1.5)
    if case["k"] == "fix":
        d["temperature"] = torch.where(torch.arange(B, device="cuda") % 4 == 0, torch.zeros_like(d["temperature"]),
                                       d["temperature"])
    d["top_p"], d["min_p"] = uni(0.5, 1.0), uni(0.0, 0.1)
    d["rep"], d["freq"], d["pres"] = uni(1.0, 1.3), uni(0.0, 0.5), uni(0.0, 0.5)
    H = case["hist"]
    if H:
        mode = mode | PENALTIES
        d["hist"] = torch.randint(0, V, (B, H), generator=g, device="cuda").to(torch.int32)
        d["bias_ids"] = _spread(g, B, NBIAS, V).to(torch.int32)
        d["bias_vals"] = torch.empty(B, NBIAS, device="cuda").uniform_(-5.0, 5.0, generator=g)
    if case["grammar"]:
        mode = mode | ssb.GRAMMAR
        W = (V + 31) // 32
        allow = torch.rand(rows, W * 32, generator=g, device="cuda") < 0.05
        top = x.float().argmax(1, keepdim=True)  # half of the rows forbid their raw maximum
        r = torch.arange(rows, device="cuda")[:, None]
        allow.scatter_(1, top, (r >> 1) % 2 == 0)
        bit = torch.ones(1, dtype=torch.int64, device="cuda") << torch.arange(32, device="cuda")
        words = torch.cat([(p.view(-1, W, 32) * bit).sum(2) for p in allow.split(64)])
        d["bitmask"] = torch.where(words >= 1 << 31, words - (1 << 32), words).to(torch.int32)
    d["mode"] = mode
    d["seed"] = torch.randint(0, 1 << 62, (B,), generator=g, device="cuda")
    d["position"] = torch.randint(0, 1 << 20, (B,), generator=g, device="cuda")
    if op == "sample_gumbel":
        d["noise"] = _exponential(g, B, V).log_()
    if verify:
        path = x.view(B, L + 1, V)
        noisy = path[:, :L].float() + torch.empty(B, L, V, device="cuda").normal_(0.0, 1.0, generator=g)
        if op == "verify":
            d["draft"] = (noisy - _exponential(g, B, L, V).log_()).argmax(2).to(torch.int32)
            d["q"] = torch.softmax(noisy, 2)
            x = path
        else:  # lists cut to 64 ids and 95 % of the mass; the path's rows among others of the tree
            val, ids = noisy.topk(min(KQ, V), 2)
            w = torch.softmax(val, 2)
            keep = (w.cumsum(2) - w) < 0.95
            q = torch.where(keep, w, 0.0)
            q = q / q.sum(2, keepdim=True)
            pick = (q.log() - _exponential(g, *q.shape).log_()).argmax(2, keepdim=True)
            d["draft"] = ids.gather(2, pick).squeeze(2).to(torch.int32)
            d["q_idx"], d["q_val"] = torch.where(keep, ids, -1).to(torch.int32), q
            Lt = L + 1 + EXTRA_ROWS
            at = torch.rand(B, Lt, generator=g, device="cuda").argsort(1)[:, :L + 1]
            tree = torch.empty(B, Lt, V, device="cuda", dtype=x.dtype).normal_(0.0, 2.0, generator=g)
            tree.scatter_(1, at[:, :, None].expand(-1, -1, V), path)
            d["row_map"] = at.to(torch.int32).contiguous()
            x = tree
    d["x"] = x
    return d


def _params(case, d):
    B, H = case["B"], case["hist"]
    t = {f: d.get(f) for f in ("mode", "temperature", "top_k", "top_p", "min_p", "rep", "freq", "pres", "bitmask",
                               "seed", "position")}
    if H:
        row = torch.arange(B + 1, device="cuda", dtype=torch.int32)
        t.update(hist_offsets=row * H, hist_ids=d["hist"].reshape(-1), bias_offsets=row * NBIAS,
                 bias_ids=d["bias_ids"].reshape(-1), bias_vals=d["bias_vals"].reshape(-1))
    return ssb.Params(B, case["V"], **t)


def prepare(case, seed):
    op, B, V, L, k_max, k_out = (case[f] for f in ("op", "B", "V", "L", "k_max", "k_out"))
    d = _inputs(case, seed)
    code = {"topk": ssb.OP_TOPK, "logprobs": ssb.OP_LOGPROBS, "process": ssb.OP_PROCESS, "verify": ssb.OP_VERIFY,
            "verify_tree": ssb.OP_VERIFY}.get(op, ssb.OP_SAMPLE)
    ws = ssb.workspace(code, B, V, L, k_max, ssb.BF16 if case["dtype"] == "bf16" else ssb.F32)
    f32 = lambda *s: torch.empty(*s, dtype=torch.float32, device="cuda")  # noqa: E731
    i32 = lambda *s: torch.empty(*s, dtype=torch.int32, device="cuda")  # noqa: E731
    # a serving loop keeps its workspace and its output buffers
    if op == "topk":
        return dict(op=op, d=d, k_max=k_max, out=dict(out_val=f32(B, k_max), out_idx=i32(B, k_max), flags=i32(B), ws=ws))
    out = dict(flags=i32(B), ws=ws)
    if op == "logprobs":
        out.update(out_idx=i32(B, k_max), out_lp=f32(B, k_max))
    elif op == "process":
        out.update(out_logits=f32(B, V), out_probs=f32(B, V))
    elif L:
        out.update(out_tokens=i32(B, L + 1), out_nacc=i32(B))
    else:
        out.update(out_token=i32(B), out_logprob=f32(B))
        if k_out:
            out.update(out_idx=i32(B, k_out), out_prob=f32(B, k_out))
    return dict(op=op, d=d, p=_params(case, d), k_max=k_max, k_out=k_out, out=out)


def run(state):
    op, d, k_max, out = state["op"], state["d"], state["k_max"], state["out"]
    x = d["x"]
    if op == "topk":
        return ssb.topk(x, d["top_k"], k_max, **out)
    p = state["p"]
    if op == "logprobs":
        return ssb.logprobs(x, p, k_max, **out)
    if op == "process":
        return ssb.process_logits(x, p, k_max, **out)[:2]
    if op == "verify":
        return ssb.verify(x, d["q"], d["draft"], p, k_max, **out)[:2]
    if op == "verify_tree":
        return ssb.verify_tree(x, d["row_map"], d["q_idx"], d["q_val"], d["draft"], p, k_max, **out)[:2]
    if op == "sample_gumbel":
        return ssb.sample_gumbel(x, p, k_max, d["noise"], **out)[:2]
    if op == "sample_full":
        return ssb.sample_full(x, p, k_max, **out)[:2]
    r = ssb.sample(x, p, k_max, k_out=state["k_out"], **out)
    return r[:2] + r[3:]


def work(case):
    """The logits once, with the bitmask, the lists and the outputs; draft probabilities and noise
    are needed at the kept ids only."""
    op, B, V, L, k_max = case["op"], case["B"], case["V"], case["L"], case["k_max"]
    rows = B * (L + 1)
    n = rows * V * (2 if case["dtype"] == "bf16" else 4)
    if case["grammar"]:
        n += rows * ((V + 31) // 32) * 4
    if case["hist"]:
        n += B * (case["hist"] * 4 + NBIAS * 8)
    if op in ("topk", "logprobs"):
        n += B * k_max * 8
    elif op == "process":
        n += B * V * 8
    elif op == "verify_tree":
        n += B * L * KQ * 8
    elif op in ("verify", "sample_gumbel"):
        n += rows * k_max * 2  # about half of the candidate bound is kept
    n += B * case["k_out"] * 8 + rows * 16
    return {"bytes": n, "flops": 2 * rows * V}


def tolerance(case):
    """Ids, counts and top-k values are exact.  Probabilities and log-probabilities come from float32
    exponentials: about one unit in the last place each."""
    if case["op"] in ("topk", "verify", "verify_tree"):
        return "exact"
    return {"rel": 4e-7, "max": 4e-6}


# ---------------------------------------------------------------------------
# The same results in 64 bits
# ---------------------------------------------------------------------------
def _processed(case, d):
    """Processed logits: each prologue step one float32 operation (taken in 64 bits and rounded);
    -inf where masked."""
    x = d["x"].float()
    if case["hist"]:
        H = d["hist"].long()
        cnt = torch.zeros_like(x).scatter_add_(1, H, torch.ones_like(H, dtype=torch.float32)).double()
        r, f, pr = (d[k].double()[:, None] for k in ("rep", "freq", "pres"))
        y = x.double()
        y = torch.where(cnt > 0, torch.where(y > 0, y / r, y * r), y).float()
        t = (f * cnt).float()
        y = torch.where(cnt > 0, (y.double() - t.double()).float(), y)
        y = torch.where(cnt > 0, (y.double() - pr).float(), y)
        x = y.scatter_add_(1, d["bias_ids"].long(), d["bias_vals"])
    if case["grammar"]:
        B, V = x.shape
        m = d["bitmask"].long() & 0xFFFFFFFF
        ok = ((m[:, :, None] >> torch.arange(32, device="cuda")) & 1).view(B, -1)[:, :V].bool()
        x = torch.where(ok, x, -math.inf)
    return x


def _uniform(d):
    """First word of Philox4x32-10 (Salmon et al., SC'11), counter (request, position, 0), key the seed."""
    u64 = np.uint64
    low = u64(0xFFFFFFFF)
    seed, pos = d["seed"].cpu().numpy().astype(u64), d["position"].cpu().numpy().astype(u64)
    c = [np.arange(len(seed)).astype(u64), pos & low, pos >> u64(32), np.zeros(len(seed), u64)]
    k = [seed & low, seed >> u64(32)]
    for _ in range(10):
        a, b = c[0] * u64(0xD2511F53), c[2] * u64(0xCD9E8D57)
        c = [(b >> u64(32)) ^ c[1] ^ k[0], b & low, (a >> u64(32)) ^ c[3] ^ k[1], a & low]
        k = [(k[0] + u64(0x9E3779B9)) & low, (k[1] + u64(0xBB67AE85)) & low]
    return torch.from_numpy((c[0].astype(np.float64) + 0.5) / 2.0 ** 32).cuda()


def exact(case, seed):
    op, k_max, V, B = case["op"], case["k_max"], case["V"], case["B"]
    if case["L"]:
        return None  # whole numbers only
    d = _inputs(case, seed)
    y = d["x"].float() if op == "topk" else _processed(case, d)
    n = min(k_max, V)
    val, ids = y.sort(dim=1, descending=True, stable=True)  # equal values: lower id first
    val, ids = val[:, :n].double(), ids[:, :n]
    rank = torch.arange(n, device="cuda")
    fill = lambda t, m, v: torch.cat([t, torch.full((B, m - t.shape[1]), v, dtype=t.dtype, device="cuda")], 1)  # noqa: E731
    if op == "topk":
        return fill(torch.where(rank < d["top_k"][:, None], val, -math.inf), k_max, -math.inf), None
    greedy = ((d["mode"] & ssb.GREEDY) != 0) | (d["temperature"] <= 0)
    tau = torch.where(greedy, 1.0, d["temperature"].double())[:, None]
    M = val[:, :1]
    if op == "logprobs":
        lse = torch.stack([((y[b].double() - M[b]) / tau[b]).logsumexp(0) for b in range(B)])[:, None]
        return None, fill((val - M) / tau - lse, k_max, -math.inf)
    k = torch.where(d["top_k"] >= 1, d["top_k"].clamp_max(n), n)[:, None] if case["k"] != "off" else torch.full((B, 1), n, device="cuda")
    z = (val - M) / tau
    w = torch.where((rank < k) & (val > -math.inf), z.exp(), 0.0)
    before = w.cumsum(1) - w
    top_p, min_p = d["top_p"].double()[:, None], d["min_p"].double()[:, None]
    cut = lambda total: (w > 0) & (before < top_p * total) & (z >= min_p.log())  # noqa: E731
    keep = cut(w.sum(1, keepdim=True))
    if op == "sample_full":
        total = torch.stack([((y[b].double() - M[b]) / tau[b]).exp().sum() for b in range(B)])[:, None]
        wide = cut(total)
        keep = torch.where(wide.sum(1, keepdim=True) < k_max, wide, keep)
    keep[:, 0] = True
    keep = torch.where(greedy[:, None], rank == 0, keep)
    P = torch.where(keep, w, 0.0)
    P = P / P.sum(1, keepdim=True)
    P = torch.where(greedy[:, None], (rank == 0).double(), P)
    if op == "process":
        full = torch.zeros(B, V, dtype=torch.float64, device="cuda").scatter_(1, ids, P)
        return y.double(), full
    if op == "sample_gumbel":
        score = torch.where(keep, z - d["noise"].gather(1, ids).double(), -math.inf)
        at = score.argmax(1, keepdim=True)
    else:
        at = (P.cumsum(1) <= _uniform(d)[:, None]).sum(1, keepdim=True)
        at = torch.minimum(at, keep.sum(1, keepdim=True) - 1)
    lp = P.gather(1, at).log().squeeze(1)
    if not case["k_out"]:
        return None, lp
    return None, lp, None, fill(P, max(n, case["k_out"]), 0.0)[:, :case["k_out"]]
