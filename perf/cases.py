"""Performance cases: the calls that a program makes into this library.

A case is a dict of plain values. ``call`` names what is called:

topk      ``indexer_topk``: one fused Indexer-TopK call. ``h``, ``d``, ``dtype``
          and ``mode`` name the scorer; ``lens`` / ``nqs`` are the key and query
          counts of the sequences (one, or several packed into one key array);
          every sequence's queries are its last positions (``causal``) or see
          all keys.
chunk     the steady state of chunked prefill: ``sample_from_topk`` over the
          previous chunk's result, then ``indexer_topk`` of the next chunk with
          that sample.
select    ``topk_select`` over a score matrix in hand.
unfused   ``indexer_scores`` and ``topk_radix``, the two-step form.
sample    ``sample_from_topk`` alone.
union     ``dsa_union`` over the top-k lists of a chunk.

Rows are requested sorted, so that the outputs have a defined order. Inputs are
drawn on the GPU by a seeded generator, with the distributions of
``paper_2607_11976_amd.workloads``: unit-variance keys and queries ("iid"), keys
and queries around a shared mean ("dsa_mean", the concentration of DSA scores),
unit vectors ("unit", "unit_self" where the queries are corpus rows), and a
mixture with outliers and duplicated keys ("adversarial").
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2607_11976_amd import litetopk as lt

DEV = "cuda"
FP8_MAX = 448.0
DTYPES = {"f32": lt.LT_F32, "bf16": lt.LT_BF16, "fp8": lt.LT_FP8_E4M3FN}

# work bounds of drawn cases: (query, key) pairs per scorer, and score elements
MAX_PAIRS = {"bf16x64": 5.0e8, "fp8x64": 2.0e9, "small": 2.0e9, "wide": 3.0e8}
MAX_SCORES = 4.0e8


def _topk(name, dtype, h, d, mode, nqs, lens, k, dist, causal=True):
    c = dict(call="topk", dtype=dtype, h=h, d=d, mode=mode, nqs=str(nqs), lens=str(lens), k=k, dist=dist,
             causal=causal)
    return dict(c, name=name) if name else c


def listed():
    return [
        # the smallest configuration: 64 queries over 4096 keys in float32
        _topk("tiny_f32", "f32", 4, 64, "dsa", 64, 4096, 256, "iid"),
        # a decode step with two speculative tokens at the end of a long context
        _topk("decode_fp8_100k", "fp8", 64, 128, "dsa", 2, 100003, 2048, "dsa_mean"),
        # a continuous batch: chunks of four sequences of ragged lengths in one call
        _topk("packed_bf16", "bf16", 64, 128, "dsa", "517,33,700,1", "20011,3001,41003,9001", 2048, "dsa_mean"),
        # a short prefill chunk at 256K context, sampling the previous chunk's result
        dict(name="chunk_bf16_256k", call="chunk", dtype="bf16", h=64, d=128, mode="dsa", nqs="128", lens="262144",
             k=2048, dist="dsa_mean", causal=True, prev=128, ns=6144),
        # the bf16 prefill chunk of 4096 queries at 128K context
        _topk("dsa_bf16_128k", "bf16", 64, 128, "dsa", 4096, 131072, 2048, "dsa_mean"),
        # the fp8 prefill chunk of 2048 queries at 1M context
        _topk("dsa_fp8_1m", "fp8", 64, 128, "dsa", 2048, 1048576, 2048, "dsa_mean"),
        # vector retrieval: 10000 queries over 4M items
        _topk("retrieval_bf16_4m", "bf16", 1, 128, "ip", 10000, 4000000, 100, "unit", causal=False),
        # passage retrieval: a batch of 64 queries over 1M 768-dimensional passages
        _topk("passages_bf16_1m", "bf16", 1, 768, "ip", 64, 1000000, 1024, "unit_self", causal=False),
        # selection from a score matrix another kernel wrote
        dict(name="select_1024x256k", call="select", nq=1024, nk=262144, k=2048, causal=True, kind="normal"),
        # dense scores and plain radix selection of a short chunk, ragged sizes
        dict(name="unfused_bf16_64k", call="unfused", dtype="bf16", h=64, d=128, mode="dsa", nqs="255", lens="65501",
             k=2048, dist="dsa_mean", causal=True),
        # the previous chunk's most frequent keys, 128K context
        dict(name="sample_1024x128k", call="sample", rows=1024, pk=2048, nk=131072, ns=6144),
        # group unions and membership masks of a chunk's lists
        dict(name="union_1024x2048", call="union", nq=1024, k=2048, nk=131072, group=8),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    call = rng.choice(["topk64", "topk64", "packed", "chunk", "small", "retrieval", "wide", "select", "unfused",
                       "sample", "union"])
    if call == "topk64":
        dt = rng.choice(["bf16", "fp8"])
        nk = _log(rng, 2048, 1048576)
        nq = max(1, min(_log(rng, 1, 4096), nk, int(MAX_PAIRS[dt + "x64"] / nk)))
        return _topk(None, dt, 64, 128, "dsa", nq, nk, min(_log(rng, 64, 4096), nk), rng.choice(["dsa_mean", "adversarial"])
                     if dt == "bf16" else "dsa_mean")
    if call == "packed":
        dt = rng.choice(["bf16", "fp8"])
        lens = [_log(rng, 512, 65536) for _ in range(rng.randint(2, 6))]
        nqs = [min(_log(rng, 1, 1024), n) for n in lens]
        return _topk(None, dt, 64, 128, "dsa", ",".join(map(str, nqs)), ",".join(map(str, lens)),
                     rng.choice([512, 1024, 2048]), "dsa_mean")
    if call == "chunk":
        dt = rng.choice(["bf16", "fp8"])
        nk = _log(rng, 16384, 1000000)
        nq = max(16, min(_log(rng, 64, 2048), int(MAX_PAIRS["bf16x64"] / 2 / nk)))
        k = rng.choice([512, 1024, 2048])
        return dict(call="chunk", dtype=dt, h=64, d=128, mode="dsa", nqs=str(nq), lens=str(nk), k=k, dist="dsa_mean",
                    causal=True, prev=max(16, nq - rng.randint(0, 15)), ns=3 * k)
    if call == "small":
        dt, h, d, mode = rng.choice([("f32", 4, 64, "dsa"), ("f32", 1, 64, "dsa"), ("f32", 1, 64, "ip"),
                                     ("bf16", 4, 128, "dsa"), ("bf16", 1, 128, "dsa")])
        nk = _log(rng, 1024, 262144)
        nq = max(1, min(_log(rng, 8, 2048), nk))
        return _topk(None, dt, h, d, mode, nq, nk, min(_log(rng, 16, 1024), nk), "iid", causal=rng.random() < 0.5)
    if call == "retrieval":
        nk = _log(rng, 65536, 4000000)
        nq = _log(rng, 16, 10000)
        return _topk(None, "bf16", 1, 128, "ip", nq, nk, _log(rng, 10, 1024), "unit", causal=False)
    if call == "wide":
        nk = _log(rng, 100000, 3000000)
        nq = max(1, min(_log(rng, 1, 128), int(MAX_PAIRS["wide"] / nk)))
        return _topk(None, "bf16", 1, 768, "ip", nq, nk, _log(rng, 16, 8192), "unit_self", causal=False)
    if call == "select":
        nk = _log(rng, 4096, 1048576)
        nq = max(1, min(_log(rng, 1, 4096), int(MAX_SCORES / nk)))
        return dict(call="select", nq=nq, nk=nk, k=min(_log(rng, 16, 4096), nk), causal=rng.random() < 0.5,
                    kind=rng.choice(["normal", "ties"]))
    if call == "unfused":
        nk = _log(rng, 4096, 262144)
        nq = max(1, min(_log(rng, 1, 1024), nk, int(MAX_SCORES / 4 / nk)))
        return dict(call="unfused", dtype=rng.choice(["bf16", "fp8"]), h=64, d=128, mode="dsa", nqs=str(nq),
                    lens=str(nk), k=_log(rng, 64, 2048), dist="dsa_mean", causal=True)
    if call == "sample":
        nk = _log(rng, 8192, 1048576)
        k = rng.choice([256, 1024, 2048])
        return dict(call="sample", rows=max(1, min(_log(rng, 1, 2048), int(1e9 / nk))), pk=k, nk=nk, ns=3 * k)
    k = rng.choice([256, 512, 1024, 2048])
    return dict(call="union", nq=_log(rng, 1, 2048), k=k, nk=_log(rng, 8192, 262144), group=rng.randint(1, 16))


# ---------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------

def _ints(text):
    return [int(v) for v in str(text).split(",")]


def _randn(g, *shape):
    return torch.randn(*shape, generator=g, device=DEV, dtype=torch.float32)


def _store(x, dtype):
    """float32 values -> storage (and per-row scales for fp8)."""
    if dtype == "f32":
        return x.contiguous(), None
    if dtype == "bf16":
        return x.to(torch.bfloat16).contiguous(), None
    amax = x.abs().amax(dim=-1)
    scale = torch.where(amax > 0, amax / FP8_MAX, torch.ones_like(amax))
    q = (x / scale.unsqueeze(-1)).clamp_(-FP8_MAX, FP8_MAX).to(torch.float8_e4m3fn)
    return q.view(torch.uint8).contiguous(), scale.contiguous()


def _keys(g, n, d, dtype, dist, mu):
    """n keys, drawn 2**20 rows at a time."""
    parts, scales = [], []
    for s in range(0, n, 1 << 20):
        m = min(1 << 20, n - s)
        x = _randn(g, m, d)
        if dist == "dsa_mean":
            x = x / math.sqrt(d) + mu
        elif dist in ("unit", "unit_self"):
            x /= x.norm(dim=1, keepdim=True)
        elif dist == "adversarial":
            x[torch.rand(m, generator=g, device=DEV) < 0.001] *= 20.0
            dup = max(1, m // 100)
            dst = torch.randperm(m, generator=g, device=DEV)[:dup]
            x[dst] = x[torch.randint(0, m, (dup,), generator=g, device=DEV)]
        p, sc = _store(x, dtype)
        parts.append(p)
        scales.append(sc)
    return (parts[0] if len(parts) == 1 else torch.cat(parts),
            None if scales[0] is None else torch.cat(scales))


def _queries(g, n, h, d, dtype, dist, mu, keys):
    if dist == "unit_self":
        pick = torch.randperm(min(keys.shape[0], 1000000), generator=g, device=DEV)[:n]
        return keys[pick].unsqueeze(1).repeat(1, h, 1).contiguous(), None
    x = _randn(g, n, h, d)
    if dist == "dsa_mean":
        x = x / math.sqrt(d) + mu
    elif dist == "unit":
        x /= x.norm(dim=2, keepdim=True)
    elif dist == "adversarial":
        x /= math.sqrt(d)
    return _store(x, dtype)


def _inputs(case, seed, extra=0):
    """Keys, queries, weights and visible ranges; `extra` more queries just
    before the last sequence's (the previous chunk)."""
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    h, d, dtype, dist = case["h"], case["d"], case["dtype"], case["dist"]
    lens, nqs = _ints(case["lens"]), _ints(case["nqs"])
    mu = _randn(g, d) / math.sqrt(d)
    keys, k_scale = _keys(g, sum(lens), d, dtype, dist, mu)
    nq = sum(nqs) + extra
    q, q_scale = _queries(g, nq, h, d, dtype, dist, mu, keys)
    w = torch.rand(nq, h, generator=g, device=DEV) if case["mode"] == "dsa" else None
    ends = starts = None
    if case["causal"]:
        e, s, base = [], [], 0
        for n, L in zip(nqs, lens):
            n += extra
            e.append(base + np.clip(L - n + np.arange(n) + 1, 0, L))
            s.append(np.full(n, base))
            base += L
        ends = torch.from_numpy(np.concatenate(e).astype(np.int32)).to(DEV)
        if len(lens) > 1:
            starts = torch.from_numpy(np.concatenate(s).astype(np.int32)).to(DEV)
    return dict(q=q, q_scale=q_scale, w=w, keys=keys, k_scale=k_scale, ends=ends, starts=starts)


def _rows(x, a, b):
    """The queries [a, b) of the inputs x."""
    cut = dict(x)
    for n in ("q", "q_scale", "w", "ends", "starts"):
        cut[n] = None if x[n] is None else x[n][a:b].contiguous()
    return cut


def _lists(g, rows, k, nk):
    """Top-k lists of consecutive queries: distinct keys per row, the popular
    ones in most rows."""
    pop = _randn(g, nk)
    out = torch.empty(rows, k, dtype=torch.int32, device=DEV)
    step = max(1, (1 << 28) // nk)
    for r in range(0, rows, step):
        m = min(step, rows - r)
        out[r:r + m] = (pop + 0.5 * _randn(g, m, nk)).topk(k, dim=1, sorted=False).indices.to(torch.int32)
    return out


def _scores(g, case):
    nq, nk = case["nq"], case["nk"]
    s = torch.empty(nq, (nk + 3) // 4 * 4, device=DEV, dtype=torch.float32)
    s.normal_(generator=g)
    if case["kind"] == "ties":
        s.mul_(64.0).round_().div_(64.0)
    ends = None
    if case["causal"]:
        ends = (torch.arange(nq, device=DEV) + (nk - nq + 1)).clamp_(0, nk).to(torch.int32)
    return s, ends


def _outputs(nq, k):
    return (torch.empty(nq, k, dtype=torch.int32, device=DEV), torch.empty(nq, k, dtype=torch.float32, device=DEV))


def prepare(case, seed):
    call, k = case["call"], case.get("k")
    st = dict(case=case)
    if call in ("topk", "chunk", "unfused"):
        x = _inputs(case, seed, case.get("prev", 0))
        nq, nk = x["q"].shape[0], x["keys"].shape[0]
        if call == "chunk":
            # the previous chunk's result, as the program has it
            p = case["prev"]
            y = _rows(x, 0, p)
            st["prev"] = lt.indexer_topk(y["q"], y["w"], y["keys"], k, y["ends"], y["q_scale"], y["k_scale"])[0]
            x = _rows(x, p, nq)
            nq -= p
            st["list"] = torch.empty(case["ns"], dtype=torch.int32, device=DEV)
            st["list_ws"] = torch.empty(lt.lt_sample_from_topk_workspace_size(nk), dtype=torch.uint8, device=DEV)
        st.update(x)
        st["out"] = _outputs(nq, k)
        if call == "unfused":
            st["scores"] = torch.empty(nq, (nk + 3) // 4 * 4, dtype=torch.float32, device=DEV)
        else:
            st["options"] = lt.make_options(sorted_output=True, visible_start=x["starts"], sample_keys=st.get("list"))
            st["workspace"] = lt.indexer_topk_workspace(nq, nk, case["h"], case["d"], DTYPES[case["dtype"]],
                                                        case["mode"], k, st["options"])
        return st
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    if call == "select":
        st["scores"], st["ends"] = _scores(g, case)
        st["out"] = _outputs(case["nq"], k)
        st["options"] = lt.make_options(sorted_output=True)
        n = lt.lt_topk_select_workspace_size(case["nq"], case["nk"], k, st["options"])
        st["workspace"] = torch.empty(n, dtype=torch.uint8, device=DEV)
    elif call == "sample":
        st["prev"] = _lists(g, case["rows"], case["pk"], case["nk"])
        st["list"] = torch.empty(case["ns"], dtype=torch.int32, device=DEV)
        st["list_ws"] = torch.empty(lt.lt_sample_from_topk_workspace_size(case["nk"]), dtype=torch.uint8, device=DEV)
    else:
        st["lists"] = _lists(g, case["nq"], k, case["nk"])
    return st


# ---------------------------------------------------------------------------
# the calls
# ---------------------------------------------------------------------------

def run(st):
    case = st["case"]
    call, k = case["call"], case.get("k")
    if call == "topk":
        return lt.indexer_topk(st["q"], st["w"], st["keys"], k, st["ends"], st["q_scale"], st["k_scale"],
                               case["mode"], st["options"], st["out"], st["workspace"])
    if call == "chunk":
        keys = lt.sample_from_topk(st["prev"], st["keys"].shape[0], case["ns"], st["list"], st["list_ws"])
        idx, scores = lt.indexer_topk(st["q"], st["w"], st["keys"], k, st["ends"], st["q_scale"], st["k_scale"],
                                      case["mode"], st["options"], st["out"], st["workspace"])
        return keys, idx, scores
    if call == "select":
        return lt.topk_select(st["scores"], k, case["nk"], st["ends"], st["options"], st["out"], st["workspace"])
    if call == "unfused":
        nk = st["keys"].shape[0]
        s = lt.indexer_scores(st["q"], st["w"], st["keys"], st["q_scale"], st["k_scale"], case["mode"], st["scores"])
        idx, scores = lt.topk_radix(s, k, nk, st["ends"], True, st["out"])
        return s[:, :nk], idx, scores
    if call == "sample":
        return lt.sample_from_topk(st["prev"], case["nk"], case["ns"], st["list"], st["list_ws"])
    return lt.dsa_union(st["lists"], case["group"])


def _pairs(case):
    """Visible (query, key) pairs."""
    total = 0
    for n, L in zip(_ints(case["nqs"]), _ints(case["lens"])):
        total += sum(max(0, min(L, L - n + t + 1)) for t in range(n)) if case["causal"] else n * L
    return total


def work(case):
    call, k = case["call"], case.get("k")
    if call in ("topk", "chunk", "unfused"):
        es = {"f32": 4, "bf16": 2, "fp8": 1}[case["dtype"]]
        nq, nk = sum(_ints(case["nqs"])), sum(_ints(case["lens"]))
        row = case["d"] * es + (4 if case["dtype"] == "fp8" else 0)
        b = nk * row + nq * case["h"] * (row + (4 if case["mode"] == "dsa" else 0)) + nq * k * 8 + 4 * nq
        pairs = _pairs(case)
        if call == "chunk":
            b += case["prev"] * k * 4 + case["ns"] * 4
        if call == "unfused":
            b += nq * nk * 4
            pairs = nq * nk
        return {"bytes": b, "flops": 2.0 * pairs * case["h"] * case["d"]}
    if call == "select":
        nq, nk = case["nq"], case["nk"]
        n = sum(max(0, min(nk, nk - nq + t + 1)) for t in range(nq)) if case["causal"] else nq * nk
        return {"bytes": 4 * n + nq * k * 8, "flops": 0.0}
    if call == "sample":
        return {"bytes": 4 * case["rows"] * case["pk"] + 4 * case["ns"], "flops": 0.0}
    nq, grp = case["nq"], case["group"]
    groups = (nq + grp - 1) // grp
    return {"bytes": 4 * nq * k + 4 * groups * (grp * k + 1) + 4 * nq * ((grp * k + 31) // 32), "flops": 0.0}


def tolerance(case):
    if case["call"] in ("select", "sample", "union"):
        return "exact"
    # scores: float32 sums in another order, about four times the distance to
    # the float64 results (bf16 and float32 1.4e-7, at most 7e-7 of one value;
    # the fp8 matrix instructions round their partial sums more coarsely:
    # 6.7e-7 and 5.5e-6). Indices: neighbours of a sorted row whose scores lie
    # within that rounding may change places (0.4% of them for bf16).
    if case["dtype"] == "fp8":
        return {"rel": 2.7e-6, "max": 2.2e-5, "differ": 0.01}
    return {"rel": 6e-7, "max": 3e-6, "differ": 0.01}


# ---------------------------------------------------------------------------
# the same results in 64 bits
# ---------------------------------------------------------------------------

def _decode(x, scale):
    if x.dtype == torch.uint8:
        return x.view(torch.float8_e4m3fn).to(torch.float64) * scale.double().unsqueeze(-1)
    return x.double()


def _exact_scores(x, mode, a, b, keys64):
    """float64 scores of queries [a, b): [b - a, nk]."""
    q = _decode(x["q"][a:b], None if x["q_scale"] is None else x["q_scale"][a:b])
    n, h, d = q.shape
    s = q.reshape(n * h, d) @ keys64.t()
    if mode == "dsa":
        s.clamp_(min=0.0)
    if h == 1:
        return s if x["w"] is None else s * x["w"][a:b].double()
    w = x["w"][a:b].double() if x["w"] is not None else torch.ones(n, h, dtype=torch.float64, device=DEV)
    return torch.bmm(w.unsqueeze(1), s.view(n, h, -1)).squeeze(1)


def _topk64(s, ends, starts, k, out_i, out_s):
    nk = s.shape[1]
    if ends is not None:
        pos = torch.arange(nk, device=DEV, dtype=torch.int32)
        hide = pos >= ends.unsqueeze(1)
        if starts is not None:
            hide |= pos < starts.unsqueeze(1)
        s = s.masked_fill(hide, -math.inf)
    v, i = s.topk(min(k, nk), dim=1, sorted=True)
    out_s[:, :v.shape[1]] = v
    out_i[:, :v.shape[1]] = torch.where(torch.isinf(v), -1, i).to(torch.int32)


def exact(case, seed):
    call, k = case["call"], case.get("k")
    if call in ("sample", "union"):
        return None  # whole numbers only
    if call == "select":
        g = torch.Generator(device=DEV)
        g.manual_seed(seed)
        s, ends = _scores(g, case)
        out_i = torch.full((case["nq"], k), -1, dtype=torch.int32, device=DEV)
        out_s = torch.full((case["nq"], k), -math.inf, dtype=torch.float64, device=DEV)
        step = max(1, (1 << 28) // case["nk"])
        for a in range(0, case["nq"], step):
            b = min(a + step, case["nq"])
            _topk64(s[a:b, :case["nk"]].double(), None if ends is None else ends[a:b], None, k, out_i[a:b], out_s[a:b])
        return out_i, out_s
    x = _inputs(case, seed, case.get("prev", 0))
    if call == "chunk":
        x = _rows(x, case["prev"], x["q"].shape[0])
    nq, nk, h = x["q"].shape[0], x["keys"].shape[0], case["h"]
    keys64 = _decode(x["keys"], x["k_scale"])
    out_i = torch.full((nq, k), -1, dtype=torch.int32, device=DEV)
    out_s = torch.full((nq, k), -math.inf, dtype=torch.float64, device=DEV)
    dense = torch.empty(nq, nk, dtype=torch.float64, device=DEV) if call == "unfused" else None
    step = max(1, (1 << 30) // (nk * h))
    for a in range(0, nq, step):
        b = min(a + step, nq)
        s = _exact_scores(x, case["mode"], a, b, keys64)
        if dense is not None:
            dense[a:b] = s
        _topk64(s, None if x["ends"] is None else x["ends"][a:b], None if x["starts"] is None else x["starts"][a:b], k,
                out_i[a:b], out_s[a:b])
    if call == "unfused":
        return dense, out_i, out_s
    return (None, out_i, out_s) if call == "chunk" else (out_i, out_s)
