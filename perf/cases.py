"""Performance cases: the calls a user of this library makes, over the range of
sizes, directions and options it serves, each through its public entry point
(``paper_2502_12085_amd.apb``).

A case is a plain dict whose ``"path"`` names the entry point:

- ``attention``  prefill attention of one host share (``attention_fwd``);
- ``compress``   ArgTop-l_p and gather of the local block (``compress_select``);
- ``scorer``     the retaining head's scores (``retaining_scores``);
- ``decode``     one host's part of a decoding step (``decode_attention``, or
  its no-allocation form);
- ``merge``      MergeScore of the hosts' partials (``merge_partials``);
- ``layer``      one host's whole transformer layer (``layer_fwd``).

``listed()`` gives the fixed cases, ``draw(rng)`` more of the same ranges,
``prepare`` what a program holds before the call (inputs, weights, output
buffers and the workspace), ``run`` one call, ``exact`` the same result in
64 bits with plain torch.
"""
from __future__ import annotations

import math

import torch

from paper_2502_12085_amd import apb

DEV = "cuda"

# Query heads, KV heads and head size of the models the workloads are shaped
# like (Llama-3.1-8B, Qwen-2.5-14B, Yi-34B), and two small ones with d = 64.
GEOMETRIES = ((32, 8, 128), (40, 8, 128), (56, 8, 128), (8, 2, 64), (4, 1, 64))
# Hidden and FFN sizes of the layer cases, by geometry.
LAYER_SIZES = {(32, 8, 128): (4096, 14336, 1024), (4, 1, 64): (256, 512, 256)}
EPS, THETA = 1e-5, 500000.0


# ------------------------------------------------------------------- cases
def _heads(g):
    return dict(n_q=g[0], n_kv=g[1], d=g[2])


def _share(hosts, host, la, lb, lp):
    return dict(hosts=hosts, host=host, la=la, lb=lb, lp=lp)


LLAMA, QWEN, TINY = _heads(GEOMETRIES[0]), _heads(GEOMETRIES[1]), _heads(GEOMETRIES[4])


def listed():
    return [
        # The smallest call: a three-token step of the tiny shape, where the
        # launches and the host path are all there is.
        dict(name="decode_tiny", path="decode", **TINY, cache=512, new=3, append=True,
             noalloc=False),
        # Every generated token after a 128K prefill over 8 hosts, last host.
        dict(name="decode_128k_token", path="decode", **LLAMA, cache=16384, new=1, append=True,
             noalloc=False),
        # The first decoding step of the same document: 64 question tokens.
        dict(name="decode_128k_question", path="decode", **LLAMA, cache=16384, new=64,
             append=True, noalloc=False),
        # A short question over an uneven split of a 256K document, on a host
        # that is not the last; called from code that cannot allocate.
        dict(name="decode_256k_ragged", path="decode", **QWEN, cache=30001, new=17, append=False,
             noalloc=True),
        # MergeScore of 8 hosts' partials of the question tokens.
        dict(name="merge_8hosts", path="merge", parts=8, rows=2048, d=128),
        # The compressor of the 128K share.
        dict(name="compress_128k", path="compress", **LLAMA, **_share(8, 7, 4096, 16384, 2048),
             zipf=False),
        # The compressor of a 1024K document over 8 hosts, tied scores: the
        # longest local block.
        dict(name="compress_1024k", path="compress", **LLAMA,
             **_share(8, 7, 8192, 131072, 16384), zipf=True),
        # The retaining head of the 32K share.
        dict(name="scorer_32k", path="scorer", **LLAMA, la=2048, lb=8192, hidden=1024),
        # Prefill attention of the last host of a 128K document (outlier K
        # channels): the headline workload.
        dict(name="attention_128k", path="attention", **LLAMA,
             **_share(8, 7, 4096, 16384, 2048), outlier=True),
        # Prefill attention of a short document (about 4K tokens over 4 hosts),
        # lengths off every tile.
        dict(name="attention_4k", path="attention", **LLAMA, **_share(4, 3, 301, 1023, 127),
             outlier=False),
        # The whole layer of the last host of a 32K document.
        dict(name="layer_32k", path="layer", **LLAMA, **_share(4, 3, 2048, 8192, 1024)),
        # The whole layer of an inner host of a short document.
        dict(name="layer_4k", path="layer", **LLAMA, **_share(4, 1, 256, 1000, 125)),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _draw_share(rng, lb_lo, lb_hi):
    lb = _log_int(rng, lb_lo, lb_hi)
    hosts = rng.choice((1, 2, 4, 8))
    la = 0 if rng.random() < 0.1 else rng.randint(max(1, lb // 16), max(1, lb // 3))
    lp = rng.randint(max(1, lb // 16), max(1, lb // 6))
    return _share(hosts, rng.randrange(hosts), la, lb, lp)


def _draw_once(rng):
    path = rng.choice(("decode", "decode", "decode", "merge", "compress", "compress", "scorer",
                       "scorer", "attention", "attention", "layer"))
    if path == "decode":
        new = 1 if rng.random() < 0.5 else _log_int(rng, 2, 256)
        return dict(path=path, **_heads(rng.choice(GEOMETRIES)), cache=_log_int(rng, 64, 65536),
                    new=new, append=rng.random() < 0.5, noalloc=rng.random() < 0.25)
    if path == "merge":
        return dict(path=path, parts=rng.randint(2, 16), rows=_log_int(rng, 4, 16384),
                    d=rng.choice((64, 128)))
    if path == "compress":
        return dict(path=path, **_heads(rng.choice(GEOMETRIES)), **_draw_share(rng, 200, 131072),
                    zipf=rng.random() < 0.3)
    if path == "scorer":
        lb = _log_int(rng, 200, 32768)
        return dict(path=path, **_heads(rng.choice(GEOMETRIES)),
                    la=rng.randint(0, max(1, lb // 3)), lb=lb,
                    hidden=rng.choice((256, 512, 1024, 1024)))
    if path == "attention":
        return dict(path=path, **_heads(rng.choice(GEOMETRIES)), **_draw_share(rng, 200, 16384),
                    outlier=rng.random() < 0.3)
    g = GEOMETRIES[0] if rng.random() < 0.8 else GEOMETRIES[4]
    return dict(path=path, **_heads(g), **_draw_share(rng, 200, 8192))


def draw(rng):
    """One more case of the same ranges, no costlier than the 128K attention."""
    most = work(next(c for c in listed() if c["name"] == "attention_128k"))["flops"]
    while True:
        c = _draw_once(rng)
        if c["path"] == "decode" and c["noalloc"]:
            # one key part has to fit the no-allocation call's scratch
            if c["n_q"] * c["new"] * (c["d"] + 1) * 4 > apb.NOALLOC_SCRATCH_BYTES:
                continue
        if work(c)["flops"] <= most:
            return c


# ------------------------------------------------------------------ inputs
def _gen(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    return g


def _normal(g, *shape, std=1.0, dtype=torch.bfloat16):
    x = torch.empty(shape, dtype=dtype, device=DEV)
    return x.normal_(0.0, std, generator=g)


def _problem(c):
    return apb.Problem(c["hosts"], c["host"], c["la"], c["lb"], c["lp"], c["n_q"], c["n_kv"],
                       c["d"])


def _kv(c, g, rows, outlier=False):
    """K and V [n_kv, rows, d] ~ N(0, 1); with ``outlier`` 2% of K's channels
    are 8 times as large, as in the 128K workload."""
    k, v = _normal(g, c["n_kv"], rows, c["d"]), _normal(g, c["n_kv"], rows, c["d"])
    if outlier:
        n = math.ceil(0.02 * c["d"])
        for h in range(c["n_kv"]):
            k[h][:, [(7 * h + 41 * j) % c["d"] for j in range(n)]] *= 8
    return k, v


def _passing(c, g, outlier=False):
    """The earlier hosts' slots [host, n_kv, l_p, d] of the passing buffers."""
    slots = [_kv(c, g, c["lp"], outlier) for _ in range(c["host"])]
    if not slots:
        return None, None
    return torch.stack([s[0] for s in slots]), torch.stack([s[1] for s in slots])


def _scores(c, g):
    shape = (c["n_kv"], c["lb"])
    if not c["zipf"]:
        return _normal(g, *shape, dtype=torch.float32)
    # whole numbers with a power-law tail: most scores are tied
    u = torch.empty(shape, device=DEV).uniform_(1e-4, 1.0, generator=g)
    return torch.floor(u.pow(-2.0))


def _scorer_weights(n_q, n_kv, d, hidden, g):
    feats = (n_q + 2 * n_kv) * d
    return dict(w1=_normal(g, hidden, feats, std=feats ** -0.5),
                b1=_normal(g, hidden, std=0.1, dtype=torch.float32),
                w2=_normal(g, n_kv, hidden, std=hidden ** -0.5, dtype=torch.float32),
                b2=_normal(g, n_kv, std=0.1, dtype=torch.float32))


def _positions(c):
    """Anchor row r at position r, local row i of this host after the anchor
    and the earlier hosts' local blocks."""
    start = c["la"] + c["host"] * c["lb"]
    return torch.cat([torch.arange(c["la"], dtype=torch.int32),
                      torch.arange(start, start + c["lb"], dtype=torch.int32)]).to(DEV)


def _layer_inputs(c, g):
    """Hidden states, weights and the earlier hosts' passed blocks.  A trained
    retaining head sets the tokens that matter apart from the rest, so l_p
    local tokens share a component that W1 picks up: which tokens are kept
    does not hang on the rounding of nearly equal scores."""
    D, inter, rh = LAYER_SIZES[(c["n_q"], c["n_kv"], c["d"])]
    n_q, n_kv, d = c["n_q"], c["n_kv"], c["d"]
    nf = (n_q + 2 * n_kv) * d
    gain = lambda: (1 + 0.1 * _normal(g, D, dtype=torch.float32)).bfloat16()  # noqa: E731
    w = dict(ln1=gain(), w_qkv=_normal(g, nf, D, std=D ** -0.5),
             w_o=_normal(g, D, n_q * d, std=(n_q * d) ** -0.5), ln2=gain(),
             w_gate=_normal(g, inter, D, std=D ** -0.5),
             w_up=_normal(g, inter, D, std=D ** -0.5),
             w_down=_normal(g, D, inter, std=inter ** -0.5))
    common = torch.sign(_normal(g, D, dtype=torch.float32))
    kept = c["la"] + torch.randperm(c["lb"], generator=g, device=DEV)[:c["lp"]]
    hidden = _normal(g, c["la"] + c["lb"], D, dtype=torch.float32)
    hidden[kept] += 2.0 * common
    hidden = hidden.bfloat16()
    s = _scorer_weights(n_q, n_kv, d, rh, g)
    seen = w["w_qkv"][(n_q + n_kv) * d:].float() @ common  # the component as V shows it
    w1 = s["w1"].float()
    w1[:, (n_q + n_kv) * d:] += 3.0 * seen / seen.square().sum()
    w.update(r_w1=w1.bfloat16(), r_b1=s["b1"], r_w2=s["w2"].abs(), r_b2=s["b2"])
    pk, pv = _passing(c, g)
    return w, hidden, pk, pv


def prepare(case, seed):
    c, g, p = case, _gen(seed), case["path"]
    bf = dict(dtype=torch.bfloat16, device=DEV)
    f32 = dict(dtype=torch.float32, device=DEV)
    if p == "decode":
        n_q, n_kv, d, new = c["n_q"], c["n_kv"], c["d"], c["new"]
        prob = apb.DecodeProblem(n_q, n_kv, d, c["cache"], new, int(c["append"]))
        s = dict(problem=prob, q=_normal(g, n_q, new, d))
        s["k_cache"], s["v_cache"] = _kv(c, g, c["cache"])
        s["k_new"], s["v_new"] = _kv(c, g, new) if c["append"] else (None, None)
        s.update(o=torch.empty(n_q, new, d, **f32), lse=torch.empty(n_q, new, **f32))
        if not c["noalloc"]:
            s["ws"] = torch.empty(apb.decode_workspace_size(prob), dtype=torch.uint8, device=DEV)
    elif p == "merge":
        P, rows, d = c["parts"], c["rows"], c["d"]
        # partials of a document cut into equal parts: O(1) values, close LSEs
        s = dict(o_parts=_normal(g, P, rows, d, dtype=torch.float32),
                 lse_parts=9.0 + _normal(g, P, rows, dtype=torch.float32),
                 o=torch.empty(rows, d, **bf), lse=torch.empty(rows, **f32))
    elif p == "compress":
        s = dict(problem=_problem(c), scores=_scores(c, g),
                 idx=torch.empty(c["n_kv"], c["lp"], dtype=torch.int32, device=DEV),
                 ok=torch.empty(c["n_kv"], c["lp"], c["d"], **bf),
                 ov=torch.empty(c["n_kv"], c["lp"], c["d"], **bf))
        s["k"], s["v"] = _kv(c, g, c["la"] + c["lb"])
    elif p == "scorer":
        rows = c["la"] + c["lb"]
        prob = apb.ScorerProblem(c["la"], c["lb"], c["n_q"], c["n_kv"], c["d"], c["hidden"])
        s = dict(problem=prob, q=_normal(g, c["n_q"], rows, c["d"]),
                 scores=torch.empty(c["n_kv"], c["lb"], **f32),
                 ws=torch.empty(apb.scorer_workspace_size(prob), dtype=torch.uint8, device=DEV))
        s["k"], s["v"] = _kv(c, g, rows)
        s.update(_scorer_weights(c["n_q"], c["n_kv"], c["d"], c["hidden"], g))
    elif p == "attention":
        rows = c["la"] + c["lb"]
        s = dict(problem=_problem(c), q=_normal(g, c["n_q"], rows, c["d"]))
        s["k"], s["v"] = _kv(c, g, rows, c["outlier"])
        s["k_pass"], s["v_pass"] = _passing(c, g, c["outlier"])
        s.update(o=torch.empty(c["n_q"], rows, c["d"], **bf),
                 lse=torch.empty(c["n_q"], rows, **f32))
    else:
        D, inter, rh = LAYER_SIZES[(c["n_q"], c["n_kv"], c["d"])]
        rows, n_kv, d = c["la"] + c["lb"], c["n_kv"], c["d"]
        prob = apb.LayerProblem(_problem(c), D, inter, rh, EPS, THETA)
        w, hidden, pk, pv = _layer_inputs(c, g)
        s = dict(problem=prob, w=w, hidden=hidden, pos=_positions(c), host=c["host"],
                 pass_k=torch.zeros(c["hosts"], n_kv, c["lp"], d, **bf),
                 pass_v=torch.zeros(c["hosts"], n_kv, c["lp"], d, **bf),
                 k_cache=torch.empty(n_kv, rows, d, **bf),
                 v_cache=torch.empty(n_kv, rows, d, **bf), out=torch.empty(rows, D, **bf),
                 ws=torch.empty(apb.layer_workspace_size(prob), dtype=torch.uint8, device=DEV))
        if pk is not None:
            s["pass_k"][:c["host"]] = pk
            s["pass_v"][:c["host"]] = pv
    s["path"] = p
    return s


# --------------------------------------------------------------------- run
def run(s):
    p = s["path"]
    if p == "decode":
        if "ws" in s:
            apb.decode_attention(s["problem"], s["q"], s["k_cache"], s["v_cache"], s["k_new"],
                                 s["v_new"], s["o"], s["lse"], s["ws"])
        else:
            apb.decode_attention_noalloc(s["problem"], s["q"], s["k_cache"], s["v_cache"],
                                         s["k_new"], s["v_new"], s["o"], s["lse"])
        return dict(o=s["o"], lse=s["lse"])
    if p == "merge":
        apb.merge_partials(s["o_parts"], s["lse_parts"], s["o"], s["lse"])
        return dict(o=s["o"], lse=s["lse"])
    if p == "compress":
        apb.compress_select(s["problem"], s["scores"], s["k"], s["v"], s["idx"], s["ok"], s["ov"])
        return dict(idx=s["idx"], k=s["ok"], v=s["ov"])
    if p == "scorer":
        apb.retaining_scores(s["problem"], s["q"], s["k"], s["v"], s["w1"], s["b1"], s["w2"],
                             s["b2"], s["scores"], s["ws"])
        return dict(scores=s["scores"])
    if p == "attention":
        apb.attention_fwd(s["problem"], s["q"], s["k"], s["v"], s["k_pass"], s["v_pass"], s["o"],
                          s["lse"])
        return dict(o=s["o"], lse=s["lse"])
    apb.layer_fwd(s["problem"], s["w"], s["hidden"], s["pos"], s["k_cache"], s["v_cache"],
                  s["pass_k"], s["pass_v"], s["out"], s["ws"])
    return dict(out=s["out"], k_cache=s["k_cache"], v_cache=s["v_cache"],
                pass_k=s["pass_k"][s["host"]], pass_v=s["pass_v"][s["host"]])


# -------------------------------------------------------------------- work
def _pairs(c):
    """Visible (query, key) pairs per query head of one host share."""
    la, lb, lp = c["la"], c["lb"], c["host"] * c["lp"]
    return la * (la + 1) / 2 + lb * (la + lp) + lb * (lb + 1) / 2


def work(case):
    c, p = case, case["path"]
    if p == "merge":
        P, rows, d = c["parts"], c["rows"], c["d"]
        return dict(bytes=P * rows * (4 * d + 4) + rows * (2 * d + 4), flops=2 * P * rows * d)
    n_q, n_kv, d = c["n_q"], c["n_kv"], c["d"]
    if p == "decode":
        new = c["new"]
        keys = c["cache"] + (new if c["append"] else 0)
        pairs = new * c["cache"] + (new * (new + 1) / 2 if c["append"] else 0)
        return dict(bytes=n_q * new * d * 2 + 4 * n_kv * keys * d + n_q * new * (4 * d + 4),
                    flops=4 * d * n_q * pairs)
    if p == "compress":
        return dict(bytes=4 * n_kv * (c["lb"] + c["lp"]) + 8 * n_kv * c["lp"] * d, flops=0)
    feats = (n_q + 2 * n_kv) * d
    if p == "scorer":
        lb, h = c["lb"], c["hidden"]
        return dict(bytes=2 * lb * feats + 2 * h * feats + 4 * h * (n_kv + 1) + 4 * n_kv * lb,
                    flops=2 * lb * feats * h + 2 * lb * h * n_kv)
    rows = c["la"] + c["lb"]
    attn = 4 * d * n_q * _pairs(c)
    passed = 4 * c["host"] * n_kv * c["lp"] * d
    if p == "attention":
        return dict(bytes=4 * n_q * rows * d + 4 * n_kv * rows * d + passed + 4 * n_q * rows,
                    flops=attn)
    D, inter, rh = LAYER_SIZES[(n_q, n_kv, d)]
    weights = 2 * (feats * D + D * n_q * d + 3 * D * inter + rh * feats + 2 * D)
    return dict(bytes=weights + 4 * rows * D + 4 * n_kv * rows * d + passed + 4 * n_kv * c["lp"] * d,
                flops=2 * rows * D * feats + 2 * rows * n_q * d * D + 6 * rows * D * inter +
                2 * c["lb"] * feats * rh + 2 * c["lb"] * rh * n_kv + attn)


# --------------------------------------------------------------- tolerance
def tolerance(case):
    """About four times the error against ``exact`` measured on these paths."""
    p = case["path"]
    if p == "compress":
        return "exact"
    if p == "scorer":
        return {"rel": 1e-5}
    return {"rel": 1e-2}


# ------------------------------------------------------------------- exact
def _attend(q, k, v, ends):
    """softmax(q k^T / sqrt(d)) v and its LSE in float64 for one head; row r
    of q sees keys 0 .. ends[r] - 1."""
    o = torch.zeros(q.shape, dtype=torch.float64, device=DEV)
    lse = torch.empty(q.shape[0], dtype=torch.float64, device=DEV)
    cols = torch.arange(k.shape[0], device=DEV)
    for r in range(0, q.shape[0], 2048):
        s = (q[r:r + 2048] @ k.T) / math.sqrt(q.shape[1])
        s.masked_fill_(cols[None, :] >= ends[r:r + 2048, None], -math.inf)
        lse[r:r + 2048] = torch.logsumexp(s, 1)
        o[r:r + 2048] = torch.exp(s.sub_(lse[r:r + 2048, None])) @ v
    return o, lse


def _attention64(c, q, k, v, pk, pv):
    la, lp = c["la"], c["host"] * c["lp"]
    rows = torch.arange(c["la"] + c["lb"], device=DEV)
    ends = torch.where(rows < la, rows, rows + lp) + 1
    o, lse = [], []
    group = c["n_q"] // c["n_kv"]
    for h in range(c["n_q"]):
        kv = h // group
        kk, vv = k[kv].double(), v[kv].double()
        if lp > 0:
            kk = torch.cat([kk[:la], pk[:c["host"], kv].double().reshape(-1, c["d"]), kk[la:]])
            vv = torch.cat([vv[:la], pv[:c["host"], kv].double().reshape(-1, c["d"]), vv[la:]])
        a, b = _attend(q[h].double(), kk, vv, ends)
        o.append(a)
        lse.append(b)
    return torch.stack(o), torch.stack(lse)


def _scores64(x, w1, b1, w2, b2):
    z = x @ w1.double().T + b1.double()
    return (torch.nn.functional.silu(z) @ w2.double().T + b2.double()).T.contiguous()


def _top64(scores, lp):
    """Indices of the l_p largest scores per head, ties to the lower index,
    ascending."""
    order = torch.argsort(scores, dim=1, descending=True, stable=True)[:, :lp]
    return torch.sort(order, dim=1).values


def _features(q, k, v, la):
    return torch.cat([t[h, la:] for t in (q, k, v) for h in range(t.shape[0])], dim=1).double()


def _rms64(h, gain):
    return h / torch.sqrt((h * h).mean(1, keepdim=True) + EPS) * gain.double()


def _layer64(c, s):
    w, n_q, n_kv, d, la = s["w"], c["n_q"], c["n_kv"], c["d"], c["la"]
    lin = lambda x, m: x @ m.double().T  # noqa: E731
    h = s["hidden"].double()
    rows = h.shape[0]
    qkv = lin(_rms64(h, w["ln1"]), w["w_qkv"]).view(rows, -1, d).transpose(0, 1)
    j = torch.arange(d // 2, device=DEV, dtype=torch.float64)
    ang = s["pos"].double()[:, None] * torch.exp(-2.0 * j / d * math.log(THETA))
    lo, hi = qkv[:n_q + n_kv, :, :d // 2], qkv[:n_q + n_kv, :, d // 2:]
    rot = torch.cat([lo * ang.cos() - hi * ang.sin(), hi * ang.cos() + lo * ang.sin()], 2)
    q, k, v = rot[:n_q], rot[n_q:], qkv[n_q + n_kv:]
    scores = _scores64(_features(q, k, v, la), w["r_w1"], w["r_b1"], w["r_w2"], w["r_b2"])
    top = _top64(scores, c["lp"]) + la
    a, _ = _attention64(c, q, k, v, s["pass_k"], s["pass_v"])
    h = h + lin(a.transpose(0, 1).reshape(rows, -1), w["w_o"])
    del a
    y = _rms64(h, w["ln2"])
    act = torch.nn.functional.silu(lin(y, w["w_gate"])) * lin(y, w["w_up"])
    h = h + lin(act, w["w_down"])
    pick = top[:, :, None].expand(-1, -1, d)
    return dict(out=h, k_cache=k, v_cache=v.contiguous(), pass_k=k.gather(1, pick),
                pass_v=v.gather(1, pick))


def exact(case, seed):
    c, s, p = case, prepare(case, seed), case["path"]
    if p == "decode":
        n_q, new, lc = c["n_q"], c["new"], c["cache"]
        k, v = s["k_cache"], s["v_cache"]
        ends = torch.full((new,), lc, device=DEV)
        if c["append"]:
            k, v = torch.cat([k, s["k_new"]], 1), torch.cat([v, s["v_new"]], 1)
            ends = ends + 1 + torch.arange(new, device=DEV)
        group = n_q // c["n_kv"]
        got = [_attend(s["q"][h].double(), k[h // group].double(), v[h // group].double(), ends)
               for h in range(n_q)]
        return dict(o=torch.stack([x[0] for x in got]), lse=torch.stack([x[1] for x in got]))
    if p == "merge":
        l64 = s["lse_parts"].double()
        lse = torch.logsumexp(l64, 0)
        return dict(o=(torch.exp(l64 - lse)[:, :, None] * s["o_parts"].double()).sum(0), lse=lse)
    if p == "compress":
        top = _top64(s["scores"].double(), c["lp"])
        pick = (top + c["la"])[:, :, None].expand(-1, -1, c["d"])
        return dict(idx=top, k=s["k"].double().gather(1, pick), v=s["v"].double().gather(1, pick))
    if p == "scorer":
        x = _features(s["q"], s["k"], s["v"], c["la"])
        return dict(scores=_scores64(x, s["w1"], s["b1"], s["w2"], s["b2"]))
    if p == "attention":
        o, lse = _attention64(c, s["q"], s["k"], s["v"], s["k_pass"], s["v_pass"])
        return dict(o=o, lse=lse)
    return _layer64(c, s)
