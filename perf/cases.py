"""The work that a user of this library has it do, as cases that can be timed and compared.

Four kinds of call sequence, each through the public binding with inputs resident in HBM:

  prefill  one attention layer of a packed batch of prompts with the observation-window importance,
           then top-k token selection: the step that bench.py times
  chunk    new tokens behind an existing KV prefix (catch-up after the first token, or one token
           per sequence while decoding); with importance over the new tokens and selection on the
           prefix, or attention alone
  select   top-k selection alone, on scores that are given
  refine   the importance of many layers aggregated, tokens selected with pooling or by sentences,
           the mask packed into its bit stream
"""
import math
from fractions import Fraction

import numpy as np
import torch

import paper_2508_09035_amd as pdd


def _ints(text):
    return [int(x) for x in str(text).split(",")]


def _cu(lengths):
    return np.concatenate([[0], np.cumsum(lengths)]).astype(np.int32)


def _keep(n, ratio):
    """k = max(1, floor(r n)), r an exact rational; 0 where nothing can be kept."""
    r = Fraction(ratio)
    return max(1, r.numerator * n // r.denominator) if n > 0 else 0


def listed():
    return [
        # one short prompt on one head: the smallest call, launches and latency
        {"name": "prefill_tiny", "kind": "prefill", "lens": "512", "hq": 1, "hkv": 1, "d": 64, "window": 32,
         "ratio": "1/2", "gain": 1.0, "heavy": False},
        # a layer of an 8B model with 4 query heads per KV head on an ordinary prompt
        {"name": "prefill_4k", "kind": "prefill", "lens": "4096", "hq": 32, "hkv": 8, "d": 128, "window": 64,
         "ratio": "3/10", "gain": 0.5, "heavy": False},
        # eight prompts of very different lengths packed into one call
        {"name": "prefill_ragged", "kind": "prefill", "lens": "2360,1384,1502,512,7898,4831,1604,3659", "hq": 32,
         "hkv": 8, "d": 128, "window": 64, "ratio": "1/2", "gain": 1.0, "heavy": False},
        # the long prompt whose refinement is the point of the method; 1 % of its keys stand out
        {"name": "prefill_32k", "kind": "prefill", "lens": "32768", "hq": 32, "hkv": 8, "d": 128, "window": 128,
         "ratio": "1/10", "gain": 1.0, "heavy": True},
        # the other head dimension
        {"name": "prefill_d64", "kind": "prefill", "lens": "3000,1111,6100", "hq": 32, "hkv": 8, "d": 64,
         "window": 64, "ratio": "1/4", "gain": 1.0, "heavy": False},
        # catch-up of four sequences, 256 new tokens each behind 8192
        {"name": "chunk_256", "kind": "chunk", "new": "256,256,256,256", "prefix": "8192,8192,8192,8192", "hq": 64,
         "hkv": 8, "d": 128, "ratio": "1/4", "gain": 1.0, "importance": True},
        # short and uneven catch-up chunks: far fewer new rows than a query tile holds
        {"name": "chunk_short", "kind": "chunk", "new": "17,64,40,5", "prefix": "5000,8192,12345,700", "hq": 32,
         "hkv": 8, "d": 128, "ratio": "1/4", "gain": 1.0, "importance": True},
        # one new token for each of eight sequences
        {"name": "chunk_decode", "kind": "chunk", "new": "1,1,1,1,1,1,1,1",
         "prefix": "2360,1384,1502,512,7898,4831,1604,3659", "hq": 32, "hkv": 8, "d": 128, "ratio": "1/4",
         "gain": 1.0, "importance": False},
        # selection in one prompt that is longer than the usual ones
        {"name": "select_long", "kind": "select", "heads": 8, "lens": "131072", "ratio": "1/10"},
        # selection for many prompts at once, at streaming size
        {"name": "select_batch", "kind": "select", "heads": 8, "lens": ",".join(["32768"] * 64), "ratio": "1/10"},
        # all layers and heads of a long prompt into one score row, whole sentences kept
        {"name": "refine_sentences", "kind": "refine", "layers": 32, "heads": 8, "lens": "32768", "ratio": "1/4",
         "reduce": True, "sentence": 24.0, "pool": 0, "pool_mode": "none"},
        # per-head scores over all layers of a few prompts, neighbours kept together by max pooling
        {"name": "refine_pooled", "kind": "refine", "layers": 32, "heads": 8, "lens": "2360,7898,4831,12001",
         "ratio": "1/4", "reduce": False, "sentence": 0.0, "pool": 7, "pool_mode": "max"},
    ]


# ---- cases of the same ranges
_HEADS = ((32, 8), (32, 8), (64, 8), (16, 2), (8, 8), (4, 2), (1, 1))


def _log(rng, lo, hi):
    """A whole number, spread evenly over its logarithm."""
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    kind = rng.choice(("prefill", "prefill", "chunk", "chunk", "select", "refine"))
    ratio = rng.choice(("1/10", "1/4", "3/10", "1/2"))
    if kind == "select":
        heads, prompts = rng.choice((1, 2, 8)), rng.choice((1, 1, 3, 16, 64))
        lens = [_log(rng, 300, 131072 if prompts <= 3 else 32768) for _ in range(prompts)]
        return {"kind": kind, "heads": heads, "lens": ",".join(map(str, lens)), "ratio": ratio}
    if kind == "refine":
        lens = [_log(rng, 300, 32768) for _ in range(rng.randint(1, 4))]
        by_sentence = rng.random() < 0.5
        return {"kind": kind, "layers": rng.randint(1, 32), "heads": rng.choice((1, 8)),
                "lens": ",".join(map(str, lens)), "ratio": ratio, "reduce": by_sentence or rng.random() < 0.3,
                "sentence": round(rng.uniform(6.0, 40.0), 1) if by_sentence else 0.0,
                "pool": 0 if by_sentence else rng.choice((3, 5, 7, 13, 33)),
                "pool_mode": "none" if by_sentence else rng.choice(("max", "avg"))}
    hq, hkv = rng.choice(_HEADS)
    d = rng.choice((64, 128, 128))
    gain = rng.choice((0.5, 1.0))
    if kind == "chunk":
        batch, importance = rng.randint(1, 8), rng.random() < 0.7
        new = [_log(rng, 1, 384) if importance else 1 for _ in range(batch)]
        prefix = [_log(rng, 100, 16384) for _ in range(batch)]
        return {"kind": kind, "new": ",".join(map(str, new)), "prefix": ",".join(map(str, prefix)), "hq": hq,
                "hkv": hkv, "d": d, "ratio": ratio, "gain": gain, "importance": importance}
    batch = rng.choice((1, 1, 2, 5, 8))
    lens = [_log(rng, 200, 16384 if batch == 1 else 8192) for _ in range(batch)]
    return {"kind": kind, "lens": ",".join(map(str, lens)), "hq": hq, "hkv": hkv, "d": d,
            "window": rng.choice((16, 32, 64, 128)), "ratio": ratio, "gain": gain, "heavy": rng.random() < 0.3}


# ---- what a user's program holds before the call
class _State:
    pass


def _device(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def _selection(s, n_rows, lens, cand, ratio):
    """Outputs of a selection among the first `cand[b]` keys of every sequence, and what describes it."""
    keep = np.array([_keep(n, ratio) for n in cand], dtype=np.int32)
    s.k_keep, s.cu_keep = _device(keep), _device(_cu(keep))
    s.total_keep = int(keep.sum())
    s.idx = torch.empty((n_rows, s.total_keep), dtype=torch.int32, device="cuda")
    s.mask = torch.empty((n_rows, sum(lens)), dtype=torch.uint8, device="cuda")


def _scores(g, *shape):
    """Importance scores: positive, a few of them far above the rest."""
    return torch.rand(shape, generator=g, device="cuda") ** 6


def _attention(case, s, g, seqlens_q, seqlens_k, chunked):
    hq, hkv, d, gain = case["hq"], case["hkv"], case["d"], case["gain"]
    tq, tk = sum(seqlens_q), sum(seqlens_k)
    normal = lambda *shape: torch.randn(shape, generator=g, device="cuda", dtype=torch.float32) * gain
    s.q = normal(tq, hq, d).bfloat16()
    k = normal(tk, hkv, d)
    if case.get("heavy"):       # 1 % of the positions shifted along one direction per KV head
        for h in range(hkv):
            u = torch.randn(d, generator=g, device="cuda")
            at = torch.randperm(tk, generator=g, device="cuda")[:max(1, tk // 100)]
            k[at, h, :] += 3.0 * u / u.norm()
    s.k = k.bfloat16()
    s.v = normal(tk, hkv, d).bfloat16()
    s.cu_q_host, s.cu_k_host = _cu(seqlens_q), _cu(seqlens_k)
    s.cu_q, s.cu_k = _device(s.cu_q_host), _device(s.cu_k_host)
    s.max_q, s.max_k = max(seqlens_q), max(seqlens_k)
    s.scale = 1.0 / math.sqrt(d)
    s.o = torch.empty_like(s.q)
    s.lse = torch.empty((hq, tq), dtype=torch.float32, device="cuda")
    s.imp = torch.empty((hkv, tk), dtype=torch.float32, device="cuda")
    desc, hold = pdd.make_desc(s.q, s.k, s.v, s.o, s.cu_q, s.cu_k, s.max_q, s.max_k, s.scale, case.get("window", 0))
    call = pdd.binding.CALL_PREFILL_ATTN_CHUNKED if chunked else pdd.binding.CALL_PREFILL_ATTN
    s.scratch = _scratch(pdd.workspace_bytes(desc, call))
    s.select_scratch = _scratch(pdd.workspace_bytes(desc, pdd.binding.CALL_SELECT_TOPK))
    del hold


def _scratch(nbytes):
    return torch.empty(nbytes, dtype=torch.uint8, device="cuda") if nbytes else None


def prepare(case, seed):
    g = torch.Generator(device="cuda").manual_seed(int(seed))
    s = _State()
    s.case = case
    if case["kind"] == "prefill":
        lens = _ints(case["lens"])
        _attention(case, s, g, lens, lens, False)
        _selection(s, case["hkv"], lens, lens, case["ratio"])
    elif case["kind"] == "chunk":
        new, prefix = _ints(case["new"]), _ints(case["prefix"])
        lens = [a + b for a, b in zip(new, prefix)]
        _attention(case, s, g, new, lens, True)
        _selection(s, case["hkv"], lens, prefix, case["ratio"])
        s.cand_b, s.cand_e = _device(np.zeros(len(new), dtype=np.int32)), _device(np.array(prefix, dtype=np.int32))
    else:
        lens = _ints(case["lens"])
        heads = case["heads"]
        s.cu_k_host = _cu(lens)
        s.cu_k, s.max_k = _device(s.cu_k_host), max(lens)
        rows = 1 if case.get("reduce") else heads
        _selection(s, rows, lens, lens, case["ratio"])
        desc = pdd.AttnDesc()
        desc.batch, desc.n_q_heads, desc.n_kv_heads, desc.head_dim = len(lens), rows, rows, 128
        desc.total_q = desc.total_k = sum(lens)
        desc.max_seqlen_q = desc.max_seqlen_k = s.max_k
        s.select_scratch = _scratch(pdd.workspace_bytes(desc, pdd.binding.CALL_SELECT_TOPK))
        if case["kind"] == "select":
            s.scores = _scores(g, heads, sum(lens))
        else:
            s.layers = _scores(g, case["layers"], heads, sum(lens))
            s.weights = torch.rand(case["layers"], generator=g, device="cuda") + 0.5
            s.scores = torch.empty((rows, sum(lens)), dtype=torch.float32, device="cuda")
            cu_bytes, s.total_bytes = pdd.pack_mask_layout(s.cu_k_host)
            s.cu_bytes = _device(cu_bytes)
            s.bits = torch.empty((rows, s.total_bytes), dtype=torch.uint8, device="cuda")
            if case["sentence"]:
                # sentences between random cuts (their lengths geometric around the case's mean), over all
                # but a fixed prefix and suffix
                rng = np.random.default_rng(seed)
                begin, ends, cu_sent = [], [], [0]
                for n in lens:
                    lo, hi = min(32, n // 8), n - min(64, n // 8)
                    count = min(8192, max(1, int((hi - lo) / case["sentence"])))
                    cuts = np.sort(rng.choice(np.arange(lo + 1, hi), size=count - 1, replace=False))
                    begin.append(lo)
                    ends.append(np.append(cuts, hi))
                    cu_sent.append(cu_sent[-1] + count)
                s.cand_b = _device(np.array(begin, dtype=np.int32))
                s.sent_end = _device(np.concatenate(ends).astype(np.int32))
                s.cu_sent = _device(np.array(cu_sent, dtype=np.int32))
                s.max_sent = max(len(e) for e in ends)
                s.budget = _device(np.array([_keep(n, case["ratio"]) for n in lens], dtype=np.int32))
                s.sent_keep = torch.empty((rows, cu_sent[-1]), dtype=torch.uint8, device="cuda")
                s.kept = torch.empty((rows, len(lens)), dtype=torch.int32, device="cuda")
    return s


# ---- one pass
def run(s):
    case = s.case
    kind = case["kind"]
    if kind == "prefill":
        pdd.prefill_attn(s.q, s.k, s.v, s.o, s.lse, s.imp, s.cu_q, s.cu_k, s.max_q, s.max_k, s.scale, case["window"],
                         s.cu_q_host, s.cu_k_host, workspace=s.scratch)
        pdd.select_topk(s.imp, s.cu_k, s.max_k, s.k_keep, s.cu_keep, s.total_keep, s.idx, s.mask, None, None,
                        s.cu_k_host, workspace=s.select_scratch)
        return {"o": s.o, "lse": s.lse, "importance": s.imp, "mask": s.mask}
    if kind == "chunk":
        pdd.prefill_attn_chunked(s.q, s.k, s.v, s.o, s.lse, s.imp if case["importance"] else None, s.cu_q, s.cu_k,
                                 s.max_q, s.max_k, s.scale, s.cu_q_host, s.cu_k_host, workspace=s.scratch)
        if not case["importance"]:
            return {"o": s.o, "lse": s.lse}
        pdd.select_topk(s.imp, s.cu_k, s.max_k, s.k_keep, s.cu_keep, s.total_keep, s.idx, s.mask, s.cand_b, s.cand_e,
                        s.cu_k_host, workspace=s.select_scratch)
        return {"o": s.o, "lse": s.lse, "importance": s.imp, "mask": s.mask}
    if kind == "select":
        pdd.select_topk(s.scores, s.cu_k, s.max_k, s.k_keep, s.cu_keep, s.total_keep, s.idx, s.mask, None, None,
                        s.cu_k_host, workspace=s.select_scratch)
        return {"indices": s.idx, "mask": s.mask}
    pdd.aggregate_scores(s.layers, s.scores, s.weights, reduce_heads=case["reduce"])
    out = {"scores": s.scores, "mask": s.mask, "bits": s.bits}
    if case["sentence"]:
        pdd.select_sentences(s.scores, s.cu_k, s.max_k, s.cu_sent, s.sent_end, s.max_sent, s.budget, pdd.SENT_MEAN,
                             s.cand_b, None, s.sent_keep, s.mask, s.kept, s.cu_k_host)
        out.update(sentences=s.sent_keep, kept=s.kept)
    else:
        mode = pdd.POOL_MAX if case["pool_mode"] == "max" else pdd.POOL_AVG
        pdd.select_topk_pooled(s.scores, s.cu_k, s.max_k, s.k_keep, s.cu_keep, s.total_keep, s.idx, s.mask,
                               case["pool"], mode, None, None, None, s.cu_k_host)
    pdd.pack_mask(s.mask, s.cu_k, s.max_k, s.cu_bytes, s.total_bytes, s.bits, s.cu_k_host)
    return out


# ---- what a pass cannot do without
def work(case):
    if case["kind"] in ("prefill", "chunk"):
        if case["kind"] == "prefill":
            nq = nk = cand = _ints(case["lens"])
            window = [min(case["window"], n) for n in nq]
        else:
            nq, cand = _ints(case["new"]), _ints(case["prefix"])
            nk = [a + b for a, b in zip(nq, cand)]
            window = nq if case["importance"] else [0] * len(nq)
        hq, hkv, d = case["hq"], case["hkv"], case["d"]
        pairs = lambda rows: sum(w * (2 * k - w + 1) // 2 for w, k in zip(rows, nk))    # the last w rows of k keys
        flops = 4 * d * hq * pairs(nq) + 2 * d * hq * pairs(window)
        # Q and O, K and V in bf16, the log-sum-exp; importance, kept indices and mask
        moved = 2 * (2 * sum(nq) * hq + 2 * sum(nk) * hkv) * d + 4 * hq * sum(nq)
        if any(window):
            moved += hkv * (4 * sum(nk) + 4 * sum(_keep(n, case["ratio"]) for n in cand) + sum(nk))
        return {"bytes": moved, "flops": flops}
    lens, heads = _ints(case["lens"]), case["heads"]
    rows, n = (1 if case.get("reduce") else heads), sum(lens)
    moved = rows * n                                                                  # mask
    if case["kind"] == "select":
        return {"bytes": moved + 4 * rows * (n + sum(_keep(x, case["ratio"]) for x in lens)), "flops": 0}
    moved += 4 * case["layers"] * heads * n + 4 * rows * n + rows * n // 8              # scores in, aggregate, bits
    if case["sentence"]:
        moved += int((4 + rows) * n / case["sentence"])
    else:
        moved += 4 * rows * sum(_keep(x, case["ratio"]) for x in lens)
    return {"bytes": moved, "flops": case["layers"] * heads * n}


def tolerance(case):
    """Selection on given scores is exact.  Attention: bf16 probabilities and a bf16 output
    (2.1e-3 to 2.4e-3 and at most 0.047 against the same path in 64 bits); a
    selection on scores that were computed may swap tokens whose scores agree to the last bits of
    their fp32 sums, two mask bytes each (a swap would move every index between the two tokens by one
    place, which is why these cases return the mask and not the indices that it determines)."""
    if case["kind"] == "select":
        return "exact"
    if case["kind"] == "refine":
        n = sum(_ints(case["lens"])) * (1 if case["reduce"] else case["heads"])
        return {"rel": 1e-6, "max": 1e-5, "differ": min(0.01, max(2e-4, 100 / n))}
    rows = case["hkv"] * sum(_ints(case["lens"] if case["kind"] == "prefill" else case["prefix"]))
    return {"rel": 1e-2, "max": 0.15, "differ": min(0.01, max(2e-4, 4 / rows))}
