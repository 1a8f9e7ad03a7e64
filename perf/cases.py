"""Workloads that stand for what a program asks of this library, with their inputs, their work and a
64-bit result to compare with.

Every case is one attention layer's call (or calls) through the public entry points, with the
buffers such a program keeps: Q, K, V or a paged cache, the output and the workspace. Fields:
  kind     prefill | dense | masked | calibrate | block_mass
  batch, hq, hkv, nb (blocks of the sequence), block, spb (sampled tokens per block)
  select   fraction | top_p, with `value`; ascending: list order
  skip     Delta as a fraction of the (shortest) sequence length, 0 for no skipping
  page     physical page size of the KV cache, 0 for contiguous K and V
  seqs     lengths in blocks of packed sequences, "" for one sequence per batch entry
"""
import math
import random

import torch

from paper_2607_25291_amd import binding as B

D = 128
_BASE = {"kind": "prefill", "batch": 1, "hq": 32, "hkv": 8, "nb": 256, "block": 128, "spb": 8,
         "select": "fraction", "value": 0.2, "ascending": False, "skip": 0.35, "page": 0, "seqs": ""}


def _case(name, **kw):
    return {"name": name, **_BASE, **kw}


def listed():
    return [
        # The smallest call: one head, 2048 tokens, 64-token blocks (a single head's probe or test).
        _case("prefill_one_head_2k", hq=1, hkv=1, nb=32, block=64, value=0.5),
        # A short prompt on a whole layer: launches and latency count.
        _case("prefill_2k", nb=16, value=0.5),
        # A layer of a 32-head, 8-KV-head model at 32K tokens.
        _case("prefill_32k", nb=256, value=0.2),
        # The same layer at 128K tokens: the long-context prefill this library exists for.
        _case("prefill_128k", nb=1024, value=0.1),
        # A wider grouped-query layer (64 / 8 heads) at 64K tokens.
        _case("prefill_wide_64k", hq=64, nb=512, value=0.15),
        # A layer without grouped queries, and a length that is no power of two.
        _case("prefill_mha_12k", hq=16, hkv=16, nb=97, value=0.3),
        # Serving: a paged cache with small pages and the mass-based stage-1 cut.
        _case("prefill_paged_top_p_8k", nb=63, select="top_p", value=0.95, page=16),
        # Serving: prompts of different lengths in one call, 64-token blocks.
        _case("prefill_packed", hq=16, hkv=4, nb=391, block=64, value=0.25,
              seqs="117,9,64,3,31,90,1,52,24"),
        # Full attention on a short or middling context, an odd number of query heads per KV head.
        _case("dense_10k", kind="dense", hq=28, hkv=4, nb=77, skip=0.0),
        # Block-sparse attention under a caller's own block mask.
        _case("masked_16k", kind="masked", nb=125, value=0.25, skip=0.0),
        # Choosing Delta for a layer: scores, lists and one walk with its margins recorded.
        _case("calibrate_16k", kind="calibrate", nb=128, value=0.2, skip=0.0),
        # Judging a selection against the exact attention mass of every block.
        _case("block_mass_8k", kind="block_mass", nb=64, skip=0.0),
    ]


def draw(rng: random.Random):
    most = work(listed()[3])["flops"]
    while True:
        kind = rng.choice(["prefill"] * 7 + ["dense", "masked", "calibrate", "block_mass"])
        hkv = rng.choice([1, 2, 4, 8, 8])
        g = rng.choice([1, 2, 3, 4, 4, 5, 7, 8])
        c = dict(_BASE, kind=kind, batch=rng.choice([1, 1, 1, 2]), hq=g * hkv, hkv=hkv,
                 block=rng.choice([64, 128, 128, 128]), spb=rng.choice([4, 8, 8, 8, 16]),
                 select=rng.choice(["fraction", "fraction", "fraction", "top_p"]),
                 ascending=rng.random() < 0.15, skip=rng.choice([0.0, 0.1, 0.35, 0.35, 0.6]))
        longest = {"prefill": 1024, "calibrate": 256, "masked": 256, "dense": 192, "block_mass": 96}[kind]
        c["nb"] = int(math.exp(rng.uniform(math.log(12), math.log(longest + 1))))
        c["value"] = round(rng.uniform(0.5, 0.95), 3) if c["select"] == "top_p" else round(
            math.exp(rng.uniform(math.log(0.05), math.log(0.6))), 3)
        if kind == "prefill":
            page = rng.choice([0, 0, 0, 16, 32, 64, 128, 256])
            if page and c["nb"] * c["block"] % page == 0:
                c["page"] = page
            if rng.random() < 0.3:
                left, parts = c["nb"], []
                while left:
                    parts.append(min(left, int(math.exp(rng.uniform(0, math.log(c["nb"]))))))
                    left -= parts[-1]
                if len(parts) <= 100:
                    c["seqs"] = ",".join(map(str, parts))
        elif kind == "calibrate":
            c["skip"] = 0.0
        elif kind == "masked":
            c["value"] = round(rng.uniform(0.05, 0.75), 3)
        if kind in ("dense", "masked", "block_mass"):
            c.update(select="fraction", ascending=False, skip=0.0, spb=8)
        w = work(c)["flops"]
        if g * c["spb"] <= 128 and _score_rows_fit(c) and w <= 0.9 * most and (w >= 1e9 or kind != "prefill"):
            return c


def _score_rows_fit(c):
    """The proxy keeps the block maxima of a query block in 160 KiB of LDS."""
    rows = c["hq"] // c["hkv"] * c["spb"]
    return 4 * rows * (c["nb"] + 1) + 5120 <= 160 * 1024


def _seqs(c):
    """(first block, blocks) of every packed sequence."""
    lens = [int(x) for x in c["seqs"].split(",")] if c["seqs"] else [c["nb"]]
    out, first = [], 0
    for n in lens:
        out.append((first, n))
        first += n
    return out


def _kept(c, n):
    """Blocks a row of n candidates keeps under the fractional budget."""
    micro = math.floor(float(torch.tensor(c["value"], dtype=torch.float32)) * 1e6 + 0.5)
    return min(max((micro * n + 999999) // 1000000, 1), n)


def work(c):
    b, L = c["block"], c["nb"] * c["block"]
    tile = 2 * b * b * D * c["batch"] * c["hq"]  # one product over a block, every query head
    qo = c["batch"] * c["hq"] * L * D * 2
    kv = c["batch"] * c["hkv"] * L * D * 2
    causal = sum(n * (n + 1) // 2 for _, n in _seqs(c))
    cells = c["batch"] * c["hkv"] * causal
    diag = tile * c["nb"]  # the half of two products above the diagonal
    if c["kind"] == "dense":
        return {"bytes": 2 * qo + 2 * kv, "flops": 2 * tile * causal - diag}
    if c["kind"] == "block_mass":
        return {"bytes": qo + kv + 4 * cells, "flops": tile * causal - diag / 2}
    if c["kind"] == "masked":
        return {"bytes": 2 * qo + 2 * kv + cells, "flops": 2 * tile * _mask_share(c) - diag}
    proxy = 2 * D * c["batch"] * c["hq"] * c["spb"] ** 2 * causal
    if c["select"] == "top_p":  # what the mass cut keeps is known only afterwards: close to the mass
        listed_ = c["value"] * causal
    else:
        listed_ = sum(_kept(c, i + 1) for _, n in _seqs(c) for i in range(n))
    # Delta scales with the shortest sequence: a packed call skips little
    computed = listed_ * (1.0 if c["seqs"] or c["skip"] == 0 else 0.5 if c["skip"] >= 0.3 else 0.8)
    out = 2 * qo + 2 * kv
    if c["kind"] == "calibrate":
        out += 9 * cells + 4 * c["batch"] * c["hq"] * listed_
    return {"bytes": out, "flops": proxy + tile * (listed_ + computed) - diag}


def _mask_share(c):
    """Blocks per KV head that the mask of _mask selects, on average."""
    nb, total = c["nb"], 0.0
    for i in range(nb):
        sure = len({0, *range(max(0, i - 2), i + 1)})
        total += sure + c["value"] * (i + 1 - sure)
    return total


# ---- inputs: sinks, a recent-token window, salient keys and queries (the structure of real
# attention maps), bf16 values; made on the GPU from the seed alone

def _ar1(gen, L, window, dev):
    """[L, D] of a unit-variance first-order autoregression with correlation length `window`."""
    rho = math.exp(-1.0 / window)
    y = torch.randn(L, D, generator=gen, device=dev)
    y[1:] *= math.sqrt(1 - rho * rho)
    s = 1
    while s < L and rho ** s > 1e-7:
        y = torch.cat([y[:s], y[s:] + rho ** s * y[:-s]])
        s *= 2
    return y


def _inputs(c, seed, dev):
    """q [B, Hq, L, D], k and v [B, Hkv, L, D], bf16."""
    gen = torch.Generator(device=dev).manual_seed(seed)
    host = random.Random(seed)
    G, L = c["hq"] // c["hkv"], c["nb"] * c["block"]
    q = torch.empty(c["batch"], c["hq"], L, D, dtype=torch.bfloat16, device=dev)
    k = torch.empty(c["batch"], c["hkv"], L, D, dtype=torch.bfloat16, device=dev)
    v = torch.randn(c["batch"], c["hkv"], L, D, generator=gen, device=dev, dtype=torch.float32).to(torch.bfloat16)
    for n in range(c["batch"]):
        for g in range(c["hkv"]):
            kk = torch.randn(L, D, generator=gen, device=dev)
            for first, _ in _seqs(c):
                kk[first * c["block"]:first * c["block"] + 4] *= 8.0
            cc = _ar1(gen, L, max(32, min(1024, L // 8)), dev)
            u = torch.randn(D, generator=gen, device=dev)
            u = 3.0 * u / u.norm()
            qq = (torch.randn(G, L, D, generator=gen, device=dev) + cc) * math.sqrt(0.5)
            kk += 0.5 * qq.mean(0)
            share = host.uniform(0.005, 0.03)
            kk += (torch.rand(L, 1, generator=gen, device=dev) < share) * u
            qq += (torch.rand(G, L, 1, generator=gen, device=dev) < 0.1) * u
            q[n, g * G:(g + 1) * G] = qq
            k[n, g] = kk
    return q, k, v


def _mask(c, seed, dev):
    """u8 [B, Hkv, nb, nb]: sink block, the last three blocks and a random share of the others."""
    gen = torch.Generator(device=dev).manual_seed(seed + 77)
    nb = c["nb"]
    i = torch.arange(nb, device=dev)[:, None]
    j = torch.arange(nb, device=dev)[None, :]
    m = torch.rand(c["batch"], c["hkv"], nb, nb, generator=gen, device=dev) < c["value"]
    return ((m | (j == 0) | (i - j < 3)) & (j <= i)).to(torch.uint8)


def _paged(c, seed, x, perm, n_pages):
    """The [n_pages, Hkv, page, D] cache holding x [B, Hkv, L, D] at the pages `perm`."""
    b, h, L, _ = x.shape
    rows = x.view(b, h, L // c["page"], c["page"], D).permute(0, 2, 1, 3, 4).reshape(-1, h, c["page"], D)
    cache = torch.zeros(n_pages, h, c["page"], D, dtype=x.dtype, device=x.device)
    cache[perm] = rows
    return cache


def _delta(c):
    return c["skip"] * min(n for _, n in _seqs(c)) * c["block"]


def prepare(case, seed):
    c, dev = case, "cuda"
    q, k, v = _inputs(c, seed, dev)
    L, nb = c["nb"] * c["block"], c["nb"]
    p = B.Problem(c["batch"], c["hq"], c["hkv"], L, D, c["block"], c["block"] // c["spb"])
    st = {"case": c, "p": p, "q": q, "k": k, "v": v}
    rows = (c["batch"], c["hkv"], nb, nb)
    if c["kind"] != "block_mass":
        st["o"] = torch.zeros_like(q)
    if c["kind"] in ("prefill", "calibrate"):
        mode = B.SELECT_TOP_P if c["select"] == "top_p" else B.SELECT_FRACTION
        st["sel"] = B.select(mode, c["value"], B.ORDER_ASCENDING if c["ascending"] else B.ORDER_KAP)
        st["skip"] = B.skip(B.SKIP_ROWMAX, _delta(c)) if c["skip"] > 0 else None
    if c["kind"] == "prefill":
        st["ws_bytes"] = B.cosa_prefill_workspace_bytes(p)
        st["ws"] = torch.zeros(st["ws_bytes"], dtype=torch.uint8, device=dev)
        if c["seqs"]:
            st["vl"] = B.varlen([f for f, _ in _seqs(c)] + [nb])
        if c["page"]:
            used = c["batch"] * L // c["page"]
            n_pages = used + used // 4 + 1
            gen = torch.Generator(device=dev).manual_seed(seed + 5)
            perm = torch.randperm(n_pages, generator=gen, device=dev)[:used]
            st["kc"], st["vc"] = (_paged(c, seed, x, perm, n_pages) for x in (k, v))
            st["table"] = perm.to(torch.int32).view(c["batch"], -1).contiguous()
            st["kv"] = B.paged_kv(st["kc"], st["vc"], st["table"], c["page"], n_pages)
            del st["k"], st["v"]
    elif c["kind"] == "calibrate":
        st["score"] = torch.zeros(rows, dtype=torch.float32, device=dev)
        st["hrm"] = torch.zeros(rows, dtype=torch.uint8, device=dev)
        st["order"] = torch.zeros(rows, dtype=torch.int32, device=dev)
        st["count"] = torch.zeros(rows[:3], dtype=torch.int32, device=dev)
        st["margin"] = torch.zeros((c["batch"], c["hq"], nb, nb), dtype=torch.float32, device=dev)
        st["n_computed"] = torch.zeros((c["batch"], c["hq"], nb), dtype=torch.int32, device=dev)
    elif c["kind"] == "masked":
        st["mask"] = _mask(c, seed, dev)
    elif c["kind"] == "block_mass":
        st["mass"] = torch.zeros(rows, dtype=torch.float32, device=dev)
    return st


def run(st):
    c, p = st["case"], st["p"]
    kind = c["kind"]
    if kind == "dense":
        B.cosa_dense_attention(p, st["q"], st["k"], st["v"], st["o"])
    elif kind == "masked":
        B.cosa_masked_attention(p, st["q"], st["k"], st["v"], st["mask"], st["o"])
    elif kind == "block_mass":
        B.cosa_block_mass(p, st["q"], st["k"], st["mass"])
        return {"mass": st["mass"]}
    elif kind == "calibrate":
        B.cosa_kap_score(p, st["q"], st["k"], st["score"], st["hrm"])
        B.cosa_kap_select_ordered(p, st["score"], st["hrm"], st["sel"], st["order"], st["count"])
        B.cosa_osk_attention(p, st["q"], st["k"], st["v"], st["order"], st["count"], st["skip"], st["o"],
                             margin_log=st["margin"], n_computed=st["n_computed"])
        return {x: st[x] for x in ("score", "hrm", "order", "count", "margin", "n_computed", "o")}
    elif "vl" in st and "kv" in st:
        B.cosa_prefill_paged_varlen(p, st["vl"], st["q"], st["kv"], st["sel"], st["skip"], st["ws"],
                                    st["ws_bytes"], st["o"])
    elif "vl" in st:
        B.cosa_prefill_varlen(p, st["vl"], st["q"], st["k"], st["v"], st["sel"], st["skip"], st["ws"],
                              st["ws_bytes"], st["o"])
    elif "kv" in st:
        B.cosa_prefill_paged(p, st["q"], st["kv"], st["sel"], st["skip"], st["ws"], st["ws_bytes"], st["o"])
    else:
        B.cosa_prefill(p, st["q"], st["k"], st["v"], st["sel"], st["skip"], st["ws"], st["ws_bytes"], st["o"])
    return {"o": st["o"]}


def tolerance(case):
    # Attention outputs are bf16 from fp32 sums over bf16 probabilities: 1.5e-3 against the 64-bit
    # result, and as much again between two orders of the sums. A listed block whose score ties with the cut, or whose margin lies on the
    # threshold, may fall on the other side: few blocks, each a visible change of its own rows.
    if case["kind"] == "block_mass":
        return {"rel": 2e-6}  # fp32 sums: 5e-8 against the 64-bit result
    return {"rel": 6e-3, "max": 0.99, "differ": 2e-3}


# ---- the 64-bit results

def _scores(c, q, k):
    """score, hrm [nb, nb] of one KV head: q [G, L, D], k [L, D], float64."""
    G, nb, spb = q.shape[0], c["nb"], c["spb"]
    s = c["block"] // spb
    score = torch.zeros(nb, nb, dtype=torch.float64, device=q.device)
    hrm = torch.zeros(nb, nb, dtype=torch.bool, device=q.device)
    for first, n in _seqs(c):
        ks = k[first * c["block"]:(first + n) * c["block"]:s]
        at = torch.arange(n * spb, device=q.device)
        total = torch.zeros(n, n, dtype=torch.float64, device=q.device)
        top = torch.zeros(n, n, dtype=torch.bool, device=q.device)
        for h in range(G):
            qs = q[h, first * c["block"]:(first + n) * c["block"]:s]
            x = (qs @ ks.T) / math.sqrt(D)
            x.masked_fill_(at[None, :] > at[:, None], -math.inf)
            beta = x.view(n * spb, n, spb).amax(2)
            mu = beta.amax(1, keepdim=True)
            total += (beta - mu).exp().view(n, spb, n).sum(1)
            top |= (beta == mu).view(n, spb, n).any(1)
        score[first:first + n, first:first + n] = total.tril()
        hrm[first:first + n, first:first + n] = top.tril()
    return score, hrm


def _lists(c, score, hrm):
    """Kept blocks of every query block, in visiting order (lists of block indices)."""
    out = []
    p = math.floor(float(torch.tensor(c["value"], dtype=torch.float32)) * 1e6 + 0.5) / 1e6
    score, hrm = score.cpu(), hrm.cpu()
    for first, n in _seqs(c):
        for i in range(first, first + n):
            s, h = score[i, first:i + 1], hrm[i, first:i + 1]
            by = torch.argsort(s, descending=True, stable=True)
            by = by[torch.argsort(h[by].to(torch.uint8), descending=True, stable=True)]
            if c["select"] == "top_p":
                cum = torch.cumsum(s[by], 0)
                kept = min(int((cum < p * float(s.sum())).sum()) + 1, len(by))
            else:
                kept = _kept(c, len(by))
            by = by[:kept] + first
            out.append((torch.sort(by).values if c["ascending"] else by).tolist())
    return out


def _walk(c, q, k, v, lists, tau):
    """o [G, L, D] and the margins of every list: Algorithm A's walk of one KV head."""
    G, b, nb = q.shape[0], c["block"], c["nb"]
    kb, vb = k.view(nb, b, D), v.view(nb, b, D)
    o = torch.zeros_like(q)
    margin = torch.zeros(G, nb, nb, dtype=torch.float64, device=q.device)
    above = torch.ones(b, b, dtype=torch.bool, device=q.device).triu(1)
    for i, lst in enumerate(lists):
        if not lst:
            continue
        K = len(lst)
        at = torch.tensor(lst, device=q.device)
        x = (q[:, i * b:(i + 1) * b].reshape(G * b, D) @ kb[at].reshape(K * b, D).T) / math.sqrt(D)
        x = x.view(G, b, K, b)
        if i in lst:
            x[:, :, lst.index(i)].masked_fill_(above, -math.inf)
        loc = x.amax(3)
        d = (loc - torch.cummax(loc, 2).values).amax(1)
        margin[:, i, :K] = d
        if tau is not None:
            x.masked_fill_((d < tau(i))[:, None, :, None], -math.inf)
        pr = torch.softmax(x.view(G * b, K * b), 1)
        o[:, i * b:(i + 1) * b] = (pr @ vb[at].reshape(K * b, D)).view(G, b, D)
    return o, margin


def exact(case, seed):
    c, dev = case, "cuda" if torch.cuda.is_available() else "cpu"
    q, k, v = _inputs(c, seed, dev)
    G, nb, b = c["hq"] // c["hkv"], c["nb"], c["block"]
    rows = (c["batch"], c["hkv"], nb, nb)
    f64 = {"dtype": torch.float64, "device": dev}
    if c["kind"] == "block_mass":
        mass = torch.zeros(rows, **f64)
        at = torch.arange(nb * b, device=dev)
        for n in range(c["batch"]):
            for h in range(c["hq"]):
                kk = k[n, h // G].double()
                for i0 in range(0, nb, 16):
                    r = slice(i0 * b, min(nb, i0 + 16) * b)
                    x = (q[n, h, r].double() @ kk.T) / math.sqrt(D)
                    x.masked_fill_(at[None, :] > at[r, None], -math.inf)
                    pr = torch.softmax(x, 1).view(-1, b, nb, b).sum((1, 3))
                    mass[n, h // G, i0:i0 + 16] += pr
        return {"mass": mass}
    o = torch.zeros(c["batch"], c["hq"], nb * b, D, dtype=torch.float32, device=dev)
    out = {"o": o}
    if c["kind"] == "calibrate":
        out = {"score": torch.zeros(rows, **f64), "hrm": None, "order": None, "count": None,
               "margin": torch.zeros(c["batch"], c["hq"], nb, nb, **f64), "n_computed": None, "o": o}
    mask = _mask(c, seed, dev).cpu() if c["kind"] == "masked" else None
    tau = None
    if c["skip"] > 0:
        delta = float(torch.tensor(_delta(c), dtype=torch.float32))
        taus = []
        for _, n in _seqs(c):
            taus += [float(torch.tensor(math.log(delta / (n * b)), dtype=torch.float32))] * n
        tau = lambda i: taus[i]  # noqa: E731
    for n in range(c["batch"]):
        for g in range(c["hkv"]):
            qq, kk, vv = q[n, g * G:(g + 1) * G].double(), k[n, g].double(), v[n, g].double()
            if c["kind"] == "dense":
                lists = [list(range(f, f + i + 1)) for f, m in _seqs(c) for i in range(m)]
            elif c["kind"] == "masked":
                lists = [torch.nonzero(mask[n, g, i]).flatten().tolist() for i in range(nb)]
            else:
                score, hrm = _scores(c, qq, kk)
                lists = _lists(c, score, hrm)
            oo, margin = _walk(c, qq, kk, vv, lists, tau)
            o[n, g * G:(g + 1) * G] = oo.to(torch.float32)
            if c["kind"] == "calibrate":
                out["score"][n, g] = score
                out["margin"][n, g * G:(g + 1) * G] = margin
    return out
