"""The work that users of this library have it do, as cases that can be prepared, run and checked.

A case is a dict of plain values:
  op        "select"  the candidate vocabulary of every row (Section 3.3, Steps 1 and 2)
            "step"    the draft step over given lists: subset logits, softmax and top-kd (Step 3)
            "chain"   both, as a drafter calls them one after the other: select, then the step over what it chose
            "dense"   the full-vocabulary projection (Section 3.1)
            "static"  a step over a fixed sub-vocabulary packed once: dense projection of the packed rows, then top-kd
            "aux"     the speculator's own log-probabilities over the whole vocabulary (Section 3.4, training)
  dtype     storage type of hidden states and weights
  rows, d, V, k, kd, d_prime   sizes (k, kd, d_prime: 0 where the operation has none)
  lists     "own": one list per row; "tree": one per row, half of it shared by all rows; "shared": one for all rows
  order     "ascending": the lists are declared sorted; "any": each is in an order of its own and nothing is declared
  padded    the lists hold padding slots (three tenths of them); for "chain": the selection runs with a score
            threshold that leaves about that many

Weights are N(0, 0.02^2), hidden states N(0, 1), lists Zipf(1.1)-distributed over the token rank without replacement,
as in the paper's kernel microbenchmark and in workloads/gen.py; everything is drawn on the GPU from the seed.
"""
from __future__ import annotations

import math
import statistics

import torch

import paper_2602_13836_amd as sv

ZIPF = 1.1
KEPT = 0.7                      # share of a padded list that holds tokens


def _case(name, op, dtype, rows, d, V, k=0, kd=0, d_prime=0, lists="own", order="ascending", padded=False):
    c = dict(op=op, dtype=dtype, rows=rows, d=d, V=V, k=k, kd=kd, d_prime=d_prime, lists=lists, order=order,
             padded=padded)
    return dict(c, name=name) if name else c


def listed():
    return [
        # the smallest call there is: one float32 row of a tiny model, selection and step; launches and host time
        _case("tiny_f32_chain", "chain", "f32", 1, 256, 8192, 512, 8, 32),
        # one token of chain drafting with a Llama-3-8B head, whole: selection, gather, softmax, top-10
        _case("chain_llama3", "chain", "bf16", 1, 4096, 128256, 8192, 10, 256),
        # the same without the selection: the indexed LM head and the draft tokens over a list at hand
        _case("step_llama3", "step", "bf16", 1, 4096, 128256, 8192, 10),
        # selection for one level of a small draft tree
        _case("tree8_select", "select", "bf16", 8, 4096, 128256, 4096, 0, 256),
        # selection for all nodes of a 60-node tree
        _case("tree60_select", "select", "bf16", 60, 4096, 128256, 4096, 0, 256),
        # the step of such a tree, each node with its own list, half of every list the same
        _case("tree60_step", "step", "bf16", 60, 4096, 128256, 4096, 10, 0, "tree", "any"),
        # eight rows that share one list under a Gemma-sized vocabulary, rows of 7.5 KiB
        _case("gemma8_step", "step", "bf16", 8, 3840, 262144, 8192, 10, 0, "shared"),
        # 16 requests x 32 tree nodes in one batch under a Qwen3-8B head: selection ...
        _case("batch512_select", "select", "bf16", 512, 4096, 151936, 8192, 0, 256),
        # ... and step
        _case("batch512_step", "step", "bf16", 512, 4096, 151936, 8192, 10),
        # full-vocabulary logits of a 60-node tree: the baseline of every step, and what verification needs
        _case("tree60_dense", "dense", "bf16", 60, 4096, 128256),
        # full-vocabulary logits of a ragged batch
        _case("batch200_dense", "dense", "bf16", 200, 4096, 128256),
        # one micro-batch of training the speculator: log-probabilities of 1024 positions over the vocabulary
        _case("train1024_aux", "aux", "bf16", 1024, 4096, 151936, 0, 0, 256),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _units(n, of):
    return max(of, n // of * of)


def draw(rng):
    while True:
        op = rng.choice(("chain", "step", "step", "select", "select", "dense", "aux", "static"))
        f32 = op in ("chain", "step", "dense", "aux") and rng.random() < 0.15
        if f32:                                        # small models only: what float32 storage is used for
            rows, d, V = _log(rng, 1, 8), _units(_log(rng, 64, 1024), 4), _log(rng, 2048, 65536)
        else:
            most = {"chain": 8, "step": 512, "select": 512, "dense": 512, "aux": 1024, "static": 64}[op]
            rows, d, V = _log(rng, 1, most), _units(_log(rng, 1024, 4096), 8), _log(rng, 16384, 262144)
        if rng.random() < 0.5:                         # published vocabularies are multiples of 64 more often than not
            V = _units(V, 64)
        d_prime = _units(max(16, d // rng.choice((8, 16))), 8) if op in ("chain", "select", "aux") else 0
        k = kd = 0
        if op not in ("dense", "aux"):
            k = _log(rng, 256, min(32768, V // 4))
            kd = rng.choice((1, 5, 8, 10, 16)) if op != "select" else 0
        lists, order, padded = "own", "ascending", False
        if op == "step":
            lists = rng.choice(("own", "tree", "shared"))
            order = rng.choice(("ascending", "ascending", "any"))
        if op in ("step", "chain"):
            padded = rng.random() < 0.15
        c = _case(None, op, "f32" if f32 else "bf16", rows, d, V, k, kd, d_prime, lists, order, padded)
        # no more than the largest listed cases do
        if rows * V * d <= 512 * 151936 * 4096 and rows * V <= 1024 * 151936 and rows * k <= 512 * 8192 * 2:
            return c


# ---- inputs


def _torch_dtype(c):
    return torch.float32 if c["dtype"] == "f32" else torch.bfloat16


def _normal(gen, rows, cols, std, dtype):
    return torch.empty((rows, cols), dtype=dtype, device="cuda").normal_(0.0, std, generator=gen)


def _zipf_lists(gen, n, V, k, without=None):
    """n lists of k different tokens each, drawn with weight rank^-1.1 (the rank is the id), in no special order."""
    race = torch.empty((n, V), dtype=torch.float32, device="cuda").exponential_(1.0, generator=gen)
    race *= torch.arange(1, V + 1, dtype=torch.float32, device="cuda") ** ZIPF
    if without is not None:
        race[:, without] = math.inf
    return torch.topk(race, k, dim=1, largest=False, sorted=False).indices


def _lists(gen, c):
    rows, V, k = c["rows"], c["V"], c["k"]
    if c["lists"] == "shared":
        idx = _zipf_lists(gen, 1, V, k)
    elif c["lists"] == "tree" and rows > 1:
        common = _zipf_lists(gen, 1, V, k // 2)
        own = _zipf_lists(gen, rows, V, k - k // 2, common[0])
        idx = torch.cat((common.expand(rows, -1), own), dim=1)
    else:
        idx = _zipf_lists(gen, rows, V, k)
    idx = idx.to(torch.int32).sort(dim=1).values
    if c["order"] == "any":
        mix = torch.rand(idx.shape, device="cuda", generator=gen).argsort(dim=1)
        idx = idx.gather(1, mix)
    if c["padded"]:
        pad = torch.rand(idx.shape, device="cuda", generator=gen) >= KEPT
        pad[:, : max(c["kd"], 1)] = False              # every row keeps enough tokens to draft from
        idx = torch.where(pad, torch.full_like(idx, -1), idx)
    return idx[0].contiguous() if c["lists"] == "shared" else idx.contiguous()


def _workspace(op, c, mode=0, k=None, V=None):
    dt = sv.SV_F32 if c["dtype"] == "f32" else sv.SV_BF16
    n = sv.workspace_bytes(op, c["rows"], c["d"], V or c["V"], c["k"] if k is None else k, c["d_prime"], c["kd"], dt, mode)
    return torch.empty(n, dtype=torch.uint8, device="cuda") if n else None


def _inputs(c, seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    dtype = _torch_dtype(c)
    s = {"h": _normal(gen, c["rows"], c["d"], 1.0, dtype)}
    if c["d_prime"]:
        s["W_down"] = _normal(gen, c["d_prime"], c["d"], 0.02, dtype)
        s["W_vocab"] = _normal(gen, c["V"], c["d_prime"], 0.02, dtype)
    if c["op"] in ("chain", "step", "dense", "static"):
        s["U"] = _normal(gen, c["V"], c["d"], 0.02, dtype)
    if c["op"] == "step":
        s["idx"] = _lists(gen, c)
    if c["op"] == "static":
        s["idx"] = _zipf_lists(gen, 1, c["V"], c["k"])[0].to(torch.int32).sort().values.contiguous()
    if c["op"] == "chain" and c["padded"]:
        # the score that seven tenths of the k best reach: the scores of a row are close to normal
        spread = 0.02 * math.sqrt(c["d_prime"]) * 0.02 * math.sqrt(c["d"])
        s["tau"] = spread * statistics.NormalDist().inv_cdf(1.0 - KEPT * c["k"] / c["V"])
    return s


def prepare(case, seed):
    """Inputs, and the output and workspace buffers that a program keeps from step to step."""
    c, s = case, _inputs(case, seed)
    rows, k, kd, V = c["rows"], c["k"], c["kd"], c["V"]

    def new(n, dtype):
        return torch.empty((rows, n), dtype=dtype, device="cuda")

    if c["op"] in ("chain", "select"):
        s["idx_out"], s["select_ws"] = new(k, torch.int32), _workspace(sv.SV_OP_SELECT, c)
    if c["op"] in ("chain", "step", "static"):
        s["logits"], s["tok"], s["prob"] = new(k, torch.float32), new(kd, torch.int32), new(kd, torch.float32)
    if c["op"] in ("chain", "step"):
        mode = sv.SV_IDX_PER_STEP if c["op"] == "step" and c["lists"] == "shared" else sv.SV_IDX_PER_ROW
        s["padded"], s["sorted"] = c["padded"], c["order"] == "ascending" and not c["padded"]
        mode |= (sv.SV_IDX_PADDED if s["padded"] else 0) | (sv.SV_IDX_SORTED if s["sorted"] else 0)
        s["step_ws"] = _workspace(sv.SV_OP_DRAFT_STEP, c, mode)
    if c["op"] == "static":
        s["packed"] = sv.pack_rows(s.pop("U"), s["idx"])
    if c["op"] == "dense":
        s["logits"] = new(V, torch.float32)
    if c["op"] == "aux":
        s["logq"], s["aux_ws"] = new(V, torch.float32), _workspace(sv.SV_OP_AUX_LOG_SOFTMAX, c)
    s["case"] = dict(c)
    return s


def run(state):
    s, c = state, state["case"]
    op = c["op"]
    out = {}
    if op in ("chain", "select"):
        sv.select(s["h"], s["W_down"], s["W_vocab"], c["k"], idx_out=s["idx_out"], ws=s["select_ws"], tau=s.get("tau"))
        out["idx"] = s["idx_out"]
    if op in ("chain", "step"):
        idx = s["idx_out"] if op == "chain" else s["idx"]
        sv.draft_step(s["h"], s["U"], idx, c["kd"], logits_out=s["logits"], tok_out=s["tok"], prob_out=s["prob"],
                      ws=s["step_ws"], padded=s["padded"], sorted_lists=s["sorted"])
    if op == "static":
        sv.dense_logits(s["h"], s["packed"], out=s["logits"])
        sv.draft_topk(s["logits"], s["idx"], c["kd"], tok_out=s["tok"], prob_out=s["prob"])
    if op in ("chain", "step", "static"):
        out.update(logits=s["logits"], tok=s["tok"], prob=s["prob"])
    if op == "dense":
        out["logits"] = sv.dense_logits(s["h"], s["U"], out=s["logits"])
    if op == "aux":
        out["logq"] = sv.aux_log_softmax(s["h"], s["W_down"], s["W_vocab"], out=s["logq"], ws=s["aux_ws"])
    return out


# ---- what a pass cannot do without, and how exact its results are


def _chance(V, k):
    """How likely each token is to be in a Zipf list of k (the exponential race's, its deadline found by bisection)."""
    w = (torch.arange(1, V + 1, dtype=torch.float64)) ** -ZIPF
    lo, hi = 0.0, 1.0
    while float((1 - torch.exp(-w * hi)).sum()) < k:
        hi *= 2
    for _ in range(60):
        mid = (lo + hi) / 2
        lo, hi = (mid, hi) if float((1 - torch.exp(-w * mid)).sum()) < k else (lo, mid)
    return 1 - torch.exp(-w * hi)


def _unique_rows(c):
    """Expected number of different rows of U that a step's lists name."""
    V, k, rows = c["V"], c["k"], c["rows"]
    if c["op"] == "chain" or c["lists"] == "shared":
        # several rows of a selection: independent sets
        n = k if c["op"] != "chain" else V * (1 - (1 - k / V) ** rows)
        return n * (KEPT if c["padded"] else 1.0)
    if c["lists"] == "tree" and rows > 1:
        p = _chance(V, k // 2)
        one = _chance(V, k - k // 2) * (1 - p)
        one = one * ((k - k // 2) / float(one.sum()))
        p, one = (p * KEPT, one * KEPT) if c["padded"] else (p, one)
        return float((1 - (1 - p) * (1 - one.clamp(max=1.0)) ** rows).sum())
    one = _chance(V, k) * (KEPT if c["padded"] else 1.0)
    return float((1 - (1 - one) ** rows).sum())


def work(case):
    c = case
    es = 4 if c["dtype"] == "f32" else 2
    rows, d, V, k, kd, dp, op = (c[x] for x in ("rows", "d", "V", "k", "kd", "d_prime", "op"))
    nbytes = rows * d * es
    flops = 0
    if dp:
        nbytes += dp * d * es + V * dp * es
        flops += 2 * rows * dp * (d + V)
    if op in ("chain", "select"):
        nbytes += rows * k * 4
    if op in ("chain", "step", "static"):
        nbytes += (k if op == "static" else _unique_rows(c)) * d * es + rows * (k + 2 * kd) * 4
        flops += 2 * rows * k * d * (KEPT if c["padded"] else 1)
    if op in ("step", "static"):
        nbytes += k * 4 * (1 if op == "static" or c["lists"] == "shared" else rows)
    if op == "dense":
        nbytes += V * d * es + rows * V * 4
        flops += 2 * rows * V * d
    if op == "aux":
        nbytes += rows * V * 4
    return {"bytes": nbytes, "flops": flops}


def tolerance(case):
    # Products of the stored values are summed in float32 whatever the storage: against 64 bits the logits are
    # 8e-8 to 4e-7 off, log-probabilities 6e-7 and draft probabilities (an exponential of a logit) up to 1.6e-6.
    # Four times that.  Ids are whole numbers that change only where two float32 sums tie or swap.
    return {"rel": 6.4e-6, "max": 1e-4, "differ": 0.01}


def _product64(x, M, chunk=16384):
    """x M^T in 64 bits, a part of M at a time."""
    out = torch.empty((x.shape[0], M.shape[0]), dtype=torch.float64, device="cuda")
    for at in range(0, M.shape[0], chunk):
        out[:, at:at + chunk] = x @ M[at:at + chunk].double().t().contiguous()
    return out


def _hidden64(c, s):
    """h' of the selector: bf16 storage rounds it to bf16."""
    hp = s["h"].double() @ s["W_down"].double().t().contiguous()
    return hp if c["dtype"] == "f32" else hp.to(torch.bfloat16).double()


def exact(case, seed):
    c = case
    if c["op"] == "select":
        return None
    s = _inputs(c, seed)
    if c["op"] == "aux":
        if c["rows"] * c["V"] > 1 << 29:
            return None
        return {"logq": torch.log_softmax(_product64(_hidden64(c, s), s["W_vocab"]), dim=1)}
    h = s["h"].double()
    if c["op"] == "dense":
        return {"logits": _product64(h, s["U"])}
    rows = c["rows"]
    if c["op"] == "chain":
        scores = _product64(_hidden64(c, s), s["W_vocab"])
        best = scores.topk(c["k"], dim=1)
        idx = torch.where(best.values >= s["tau"], best.indices, -1) if "tau" in s else best.indices
    else:
        idx = s["idx"].long()
        idx = idx.expand(rows, -1) if idx.dim() == 1 else idx
    if c["op"] in ("step", "static") and s["idx"].dim() == 1:
        logits = _product64(h, s["U"][s["idx"].long().clamp(min=0)])
    else:
        logits = _product64(h, s["U"]).gather(1, idx.clamp(min=0))
    logits = logits.masked_fill(idx < 0, -math.inf)
    prob = torch.softmax(logits, dim=1).topk(c["kd"], dim=1).values
    out = {"logits": None if c["op"] == "chain" else logits, "tok": None, "prob": prob}
    return dict(out, idx=None) if c["op"] == "chain" else out
