"""The work a user of libstreamindex has it do, as measurable cases.

Each case is one call of one public entry point on inputs that live on the GPU:

  indexer      si_indexer_topk: scores of every legal (query, key) pair and the k best keys per query
  attention    si_sparse_attention: the consumer of the index lists
  from_scores  si_topk_from_scores: selection alone, on scores the caller has
  score_tile   si_score_tile: dense scores alone

Sizes are those of the evaluation shapes (64 heads of 128, one compressed key per 4 positions, k 512
or 1024, causal block mask), of the parity cases (few heads, heads of 32 or 64, batches, ragged sizes)
and of the calls a serving loop makes: decoding one or a few positions of each request against that
request's whole cache, where every key is legal.
"""
import math

import torch

import paper_2605_02568_amd as P

DEV = "cuda:0"
NONE, CAUSAL = P.SI_MASK_NONE, P.SI_MASK_CAUSAL_BLOCK


def _indexer(name, B, S, H, D, T, m, k, mask):
    return {"name": name, "op": "indexer", "B": B, "S": S, "H": H, "D": D, "T": T, "m": m, "k": k, "mask": mask}


def _attention(name, B, S, H, D, T, m, k, n_win, mask):
    return {"name": name, "op": "attention", "B": B, "S": S, "H": H, "D": D, "T": T, "m": m, "k": k,
            "n_win": n_win, "mask": mask}


def listed():
    return [
        # the smallest whole call: the parity configuration, bound by launches and latency
        _indexer("tiny", 1, 1024, 4, 32, 256, 4, 16, NONE),
        # prefill of a short prompt: most of the work is per row, not per key
        _indexer("prefill_4k", 1, 4096, 64, 128, 1024, 4, 512, CAUSAL),
        # a batch of ragged prompts with another head shape and a small k
        _indexer("prefill_ragged", 2, 8191, 33, 64, 2047, 4, 300, CAUSAL),
        # prefill of an ordinary long prompt
        _indexer("prefill_64k", 1, 65536, 64, 128, 16384, 4, 512, CAUSAL),
        # the largest: prefill of a 1M-position context
        _indexer("prefill_1m", 1, 1048576, 64, 128, 262144, 4, 1024, CAUSAL),
        # lists longer than the single-pass schedule takes, one key per position
        _indexer("wide_list", 1, 16384, 64, 128, 16384, 1, 4096, CAUSAL),
        # one new position of one request against a 1M-position cache
        _indexer("decode_1m", 1, 1, 64, 128, 262144, 4, 1024, NONE),
        # two new positions of each of 32 requests against caches of 64k positions
        _indexer("decode_batch", 32, 2, 64, 128, 16411, 4, 512, NONE),
        # the consumer of the lists in prefill and in decode
        _attention("attention_prefill", 1, 16384, 64, 128, 4096, 4, 512, 128, CAUSAL),
        _attention("attention_decode", 32, 1, 64, 128, 65536, 4, 1024, 128, NONE),
        # selection alone, on ragged rows
        {"name": "from_scores", "op": "from_scores", "R": 2048, "n": 32771, "k": 512, "c_T": 4096, "ragged": True},
        # dense scores alone
        {"name": "score_tile", "op": "score_tile", "B": 1, "S": 2048, "H": 64, "D": 128, "T": 16384, "c_S": 2048,
         "c_T": 16384},
    ]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    kind = rng.choice(["prefill", "prefill", "decode", "decode", "attention", "attention_decode", "from_scores",
                       "score_tile", "wide"])
    H, D = rng.choice([(64, 128), (64, 128), (64, 128), (rng.randint(1, 64), rng.choice([32, 64, 128]))])
    if kind == "prefill":
        S, m = _log_int(rng, 500, 200000), rng.choice([1, 2, 4, 4, 4, 8])
        S = min(S, int(131072 * math.sqrt(m)))
        B = rng.randint(1, 3) if S < 20000 else 1
        return _drop(_indexer("", B, S, H, D, max(1, S // m), m, _log_int(rng, 16, 2048), rng.choice([CAUSAL, CAUSAL, CAUSAL, NONE])
                              if S < 30000 else CAUSAL))
    if kind == "decode":
        B, S, T = _log_int(rng, 1, 128), rng.choice([1, 1, 1, 2, 4]), _log_int(rng, 1000, 262144)
        B = max(1, min(B, 12000000 // T))
        return _drop(_indexer("", B, S, H, D, T, 4, _log_int(rng, 64, 2048), NONE))
    if kind == "wide":
        S = _log_int(rng, 2000, 20000)
        return _drop(_indexer("", 1, S, H, D, S, 1, _log_int(rng, 2049, 4096), CAUSAL))
    if kind == "attention":
        S, m, D = _log_int(rng, 200, 20000), 4, rng.choice([64, 128, 128])
        return _drop(_attention("", rng.randint(1, 2), S, H, D, max(1, S // m), m, _log_int(rng, 16, 1024),
                                rng.choice([0, 64, 128]), CAUSAL))
    if kind == "attention_decode":
        B, T, D = _log_int(rng, 1, 128), _log_int(rng, 1000, 100000), rng.choice([64, 128, 128])
        return _drop(_attention("", B, rng.choice([1, 1, 2]), H, D, T, 4, _log_int(rng, 64, 2048),
                                rng.choice([0, 128]), NONE))
    if kind == "from_scores":
        n = _log_int(rng, 500, 262144)
        R = max(1, min(_log_int(rng, 1, 8192), 100000000 // n))
        return {"op": "from_scores", "R": R, "n": n, "k": _log_int(rng, 16, 4096), "c_T": rng.choice([1024, 4096, 8192, 16384]),
                "ragged": rng.random() < 0.5}
    S, T = _log_int(rng, 64, 4096), _log_int(rng, 500, 20000)
    return {"op": "score_tile", "B": rng.randint(1, 2), "S": S, "H": H, "D": D, "T": T, "c_S": S, "c_T": T}


def _drop(case):
    return {key: v for key, v in case.items() if key != "name"}


def _legal(case):
    """Legal keys of each query position (position = row)."""
    S, T = case["S"], case["T"]
    if case["mask"] == NONE:
        return torch.full((S,), T, dtype=torch.int64)
    return torch.clamp((torch.arange(S, dtype=torch.int64) + 1) // case["m"], max=T)


# ---------------------------------------------------------------------------------- inputs
def _normal(gen, shape, dtype, scale=1.0):
    out = torch.empty(shape, dtype=dtype, device=DEV)
    flat = out.view(-1)
    step = 1 << 28  # bounds the float32 temporary
    for i in range(0, flat.numel(), step):
        part = torch.randn(min(step, flat.numel() - i), generator=gen, device=DEV, dtype=torch.float32)
        flat[i:i + step] = part.mul_(scale).to(dtype)
    return out


def _lists(gen, case):
    """Index lists as the indexer writes them: distinct legal keys in no particular index order, pads last."""
    B, S, T, k = case["B"], case["S"], case["T"], case["k"]
    legal = _legal(case).to(DEV)
    out = torch.full((B, S, k), -1, dtype=torch.int32, device=DEV)
    kk = min(k, T)
    step = max(1, (1 << 26) // T)
    for b in range(B):
        for s in range(0, S, step):
            e = min(S, s + step)
            r = torch.rand((e - s, T), generator=gen, device=DEV)
            r.masked_fill_(torch.arange(T, device=DEV)[None, :] >= legal[s:e, None], -1.0)
            v, i = torch.topk(r, kk, dim=1)
            out[b, s:e, :kk] = torch.where(v >= 0, i, -1).to(torch.int32)
    return out


def prepare(case, seed):
    gen = torch.Generator(device=DEV)
    gen.manual_seed(seed)
    op = case["op"]
    st = {"case": case}
    if op == "from_scores":
        R, n, k = case["R"], case["n"], case["k"]
        st["scores"] = _normal(gen, (R, n), torch.float32)
        st["legal"] = None
        if case["ragged"]:
            st["legal"] = torch.randint(max(1, n // 4), n + 1, (R,), generator=gen, device=DEV, dtype=torch.int32)
        st["idx"] = torch.empty((R, k), dtype=torch.int32, device=DEV)
        st["score"] = torch.empty((R, k), dtype=torch.float32, device=DEV)
        nbytes = P.si_workspace_bytes(1, R, 1, 32, n, k, R, case["c_T"])
        st["ws"] = torch.empty(nbytes, dtype=torch.uint8, device=DEV)
        return st
    B, S, H, D, T = (case[x] for x in ("B", "S", "H", "D", "T"))
    st["q"] = _normal(gen, (B, S, H, D), torch.bfloat16)
    st["K"] = _normal(gen, (B, T, D), torch.bfloat16)
    if op == "attention":
        st["idx"] = _lists(gen, case)
        st["out"] = torch.empty((B, S, H, D), dtype=torch.float32, device=DEV)
        return st
    st["w"] = _normal(gen, (B, S, H), torch.float32, 1.0 / math.sqrt(H))
    if op == "score_tile":
        st["tile"] = torch.empty((B, case["c_S"], case["c_T"]), dtype=torch.float32, device=DEV)
        return st
    k = case["k"]
    st["idx"] = torch.empty((B, S, k), dtype=torch.int32, device=DEV)
    st["score"] = torch.empty((B, S, k), dtype=torch.float32, device=DEV)
    nbytes = P.si_fused_workspace_bytes(B, S, H, D, T, k)
    if nbytes == 0:  # k beyond the single-pass schedule: tiles planned for a budget of 2 GiB
        nbytes = P.si_plan_tiles(B, S, H, D, T, case["m"], k, case["mask"], 2 << 30)[2]
    st["ws"] = torch.empty(nbytes, dtype=torch.uint8, device=DEV)
    return st


# ---------------------------------------------------------------------------------- the pass
def run(state):
    case = state["case"]
    op = case["op"]
    if op == "indexer":
        P.si_indexer_topk(state["q"], state["K"], state["w"], case["m"], case["k"], case["mask"], state["idx"],
                          state["score"], state["ws"])
        return {"idx": state["idx"], "score": state["score"]}
    if op == "attention":
        P.si_sparse_attention(state["q"], state["K"], state["idx"], case["m"], case["mask"], case["n_win"],
                              1.0 / math.sqrt(case["D"]), state["out"])
        return {"out": state["out"]}
    if op == "from_scores":
        P.si_topk_from_scores(state["scores"], state["legal"], case["k"], case["c_T"], state["idx"], state["score"],
                              state["ws"])
        return {"idx": state["idx"], "score": state["score"]}
    P.si_score_tile(state["q"], state["K"], state["w"], 1, NONE, 0, 0, case["c_S"], case["c_T"], state["tile"])
    return {"tile": state["tile"]}


def work(case):
    op = case["op"]
    if op == "from_scores":
        R, n, k = case["R"], case["n"], case["k"]
        # legal lengths are uniform over n/4 .. n where they are ragged
        return {"bytes": R * n * 4 * (0.625 if case["ragged"] else 1.0) + R * k * 8, "flops": 0}
    B, S, H, D, T = (case[x] for x in ("B", "S", "H", "D", "T"))
    inputs = B * S * H * D * 2 + B * T * D * 2
    if op == "score_tile":
        return {"bytes": inputs + B * S * H * 4 + B * S * T * 4, "flops": 2 * B * S * T * H * D}
    legal = _legal(case)
    if op == "attention":
        win = torch.clamp(legal, max=case["n_win"])
        listed_keys = torch.clamp(legal, max=case["k"])
        # keys that the window already holds are listed with the probability that a random legal key is one
        both = listed_keys.double() * win / torch.clamp(legal, min=1)
        union = B * float((listed_keys + win - both).sum())
        rows = min(B * T, union)  # key rows that are read at all
        nbytes = B * S * H * D * 2 + rows * D * 2 + B * S * case["k"] * 4 + B * S * H * D * 4
        return {"bytes": nbytes, "flops": 4 * union * H * D}
    return {"bytes": inputs + B * S * H * 4 + B * S * case["k"] * 8, "flops": 2 * B * int(legal.sum()) * H * D}


def tolerance(case):
    op = case["op"]
    if op == "from_scores":
        return "exact"
    # four times the largest difference from exact() seen over the listed and twenty drawn cases
    if op == "attention":  # weights of 16 mantissa bits: 1.2e-6 .. 2.1e-6, largest 5e-5
        return {"rel": 8e-6, "max": 2e-4}
    if op == "score_tile":  # 32-bit sums: 1.0e-7, largest 1e-6
        return {"rel": 4e-7, "max": 4e-6}
    # two keys whose scores differ by less than the rounding of a 32-bit sum may change places: 3.2e-4
    return {"rel": 4e-7, "max": 4e-6, "differ": 1.3e-3}


# ---------------------------------------------------------------------------------- in 64 bits
def _scores64(q, Kt, w):
    """q [r,H,D], Kt [D,T], w [r,H] -> [r,T], all float64."""
    r, H, D = q.shape
    x = (q.reshape(r * H, D) @ Kt).clamp_(min=0.0).view(r, H, -1)
    return x.mul_(w[:, :, None]).sum(dim=1)


def _best(scores, legal, k):
    """Best first, the smaller index first among equals, pads last."""
    n = scores.shape[1]
    s = scores.masked_fill(torch.arange(n, device=DEV)[None, :] >= legal[:, None], -math.inf)
    v, i = torch.sort(s, dim=1, descending=True, stable=True)
    kk = min(k, n)
    idx = torch.full((s.shape[0], k), -1, dtype=torch.int32, device=DEV)
    val = torch.full((s.shape[0], k), -math.inf, dtype=torch.float64, device=DEV)
    live = torch.arange(kk, device=DEV)[None, :] < legal[:, None]
    idx[:, :kk] = torch.where(live, i[:, :kk], -1).to(torch.int32)
    val[:, :kk] = torch.where(live, v[:, :kk], -math.inf)
    return idx, val


def exact(case, seed):
    op = case["op"]
    if op != "from_scores" and case["B"] * case["S"] * case["T"] * case["H"] > 1.5e11 and op != "attention":
        return None  # over 20 seconds
    st = prepare(case, seed)
    if op == "from_scores":
        R, n, k = case["R"], case["n"], case["k"]
        legal = st["legal"] if st["legal"] is not None else torch.full((R,), n, device=DEV)
        idx = torch.empty((R, k), dtype=torch.int32, device=DEV)
        val = torch.empty((R, k), dtype=torch.float64, device=DEV)
        step = max(1, (1 << 26) // n)
        for r in range(0, R, step):
            idx[r:r + step], val[r:r + step] = _best(st["scores"][r:r + step].double(), legal[r:r + step], k)
        return {"idx": idx, "score": val}
    B, S, H, D, T = (case[x] for x in ("B", "S", "H", "D", "T"))
    if op == "attention":
        return {"out": _attention64(st)}
    step = max(1, (1 << 28) // (H * T))
    if op == "score_tile":
        tile = torch.empty((B, S, T), dtype=torch.float64, device=DEV)
    else:
        legal = _legal(case).to(DEV)
        idx = torch.empty((B, S, case["k"]), dtype=torch.int32, device=DEV)
        val = torch.empty((B, S, case["k"]), dtype=torch.float64, device=DEV)
    for b in range(B):
        Kt = st["K"][b].double().t().contiguous()
        for s in range(0, S, step):
            e = min(S, s + step)
            sc = _scores64(st["q"][b, s:e].double(), Kt, st["w"][b, s:e].double())
            if op == "score_tile":
                tile[b, s:e] = sc
            else:
                idx[b, s:e], val[b, s:e] = _best(sc, legal[s:e], case["k"])
    return {"tile": tile} if op == "score_tile" else {"idx": idx, "score": val}


def _attention64(st):
    case = st["case"]
    B, S, H, D, T, n_win = (case[x] for x in ("B", "S", "H", "D", "T", "n_win"))
    legal = _legal(case).to(DEV)
    out = torch.empty((B, S, H, D), dtype=torch.float64, device=DEV)
    step = max(1, (1 << 26) // ((case["k"] + n_win) * D))
    for b in range(B):
        K = st["K"][b].double()
        for s in range(0, S, step):
            e = min(S, s + step)
            L = legal[s:e, None]
            first = (L - n_win).clamp(min=0)
            listed_keys = st["idx"][b, s:e].long()
            ok = (listed_keys >= 0) & ~((listed_keys >= first) & (listed_keys < L))
            window = first + torch.arange(n_win, device=DEV)[None, :]
            keys = torch.cat([listed_keys.clamp(min=0), window.clamp(max=T - 1)], dim=1)
            ok = torch.cat([ok, window < L], dim=1)
            rows = K[keys]                                                     # [r, U, D]
            x = torch.matmul(st["q"][b, s:e].double(), rows.transpose(1, 2).contiguous()) / math.sqrt(D)
            x.masked_fill_(~ok[:, None, :], -math.inf)
            top = x.amax(dim=2, keepdim=True)
            p = torch.exp(x - torch.where(torch.isfinite(top), top, torch.zeros_like(top)))
            total = p.sum(dim=2, keepdim=True)
            out[b, s:e] = torch.matmul(p, rows) / torch.where(total > 0, total, torch.ones_like(total))
    return out
