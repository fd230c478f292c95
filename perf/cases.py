"""What a user of this framework has it do, as cases that can be timed.

Twelve listed cases cover the public entry points over the range of sizes in
which they are used: single tokens, short layers, corpus and long-context
encodes, the query-time path, retrieval, injection and the consolidation of
semantic states.  `draw` gives more cases of the same ranges.  Inputs follow
the recipe of the package's synthetic workloads (x, z ~ N(0, 1), dt =
softplus(N(mu, sigma)), A ~ U[1, 16], B, C ~ N(0, 1/N), unit-norm keys and
queries, part of the queries near a key) and are drawn on the device.

Kinds of cases:

  scan        one scan through precog_scan_encode with the caller's buffers
  encode      the same through the allocating wrapper
  trajectory  the scan that keeps every `every`-th state
  complex     the scan with a complex diagonal A
  query       exact top-1, injection and query prefill in one call
  topk        exact top-k over an index
  fuse        composition of episodic and corpus candidates, plus the
              session's semantic state
  smc         routing of chunks, then consolidation of their states
"""
from __future__ import annotations

import math

import torch

from paper_2608_02560_amd import precog as P

DEV = "cuda"
_T = {"f32": torch.float32, "bf16": torch.bfloat16, "f16": torch.float16}
_SIZE = {"f32": 4, "bf16": 2, "f16": 2}


def listed():
    return [
        # one token of 8 running sessions, state in and out: the smallest
        # call there is, nothing but latency
        dict(name="session_step", kind="scan", B=8, L=1, D=2048, N=16, io="bf16", out="bf16", st="f32",
             y=True, z=True, h0=True, mu=-2.0, sigma=0.5),
        # one fp32 layer over one 512-token chunk (the chunk length of the
        # offline index), everything in 32 bits
        dict(name="layer_f32", kind="scan", B=1, L=512, D=128, N=16, io="f32", out="f32", st="f32",
             y=True, z=True, h0=False, mu=-2.0, sigma=0.5),
        # a few documents of an odd length through an odd number of channels,
        # 32-bit, ungated, from injected states
        dict(name="ragged_f32", kind="encode", B=5, L=1237, D=1000, N=16, io="f32", out="f32", st="f32",
             y=True, z=False, h0=True, mu=-2.0, sigma=0.5),
        # offline indexing of 64 contexts of 3,000 tokens with outputs: the
        # largest ordinary encode
        dict(name="encode_corpus", kind="encode", B=64, L=3000, D=2048, N=16, io="bf16", out="bf16", st="f16",
             y=True, z=True, h0=False, mu=-2.0, sigma=0.5),
        # part of one layer of the large corpus: 64 states a channel, final
        # states only
        dict(name="corpus_states_n64", kind="encode", B=96, L=3000, D=1536, N=64, io="bf16", out="bf16", st="f16",
             y=False, z=False, h0=False, mu=-3.0, sigma=1.0),
        # two long contexts: too few channels to fill the GPU without
        # cutting time
        dict(name="long_context", kind="encode", B=2, L=65536, D=2048, N=16, io="bf16", out="bf16", st="f16",
             y=True, z=True, h0=False, mu=-2.0, sigma=0.5),
        # conversation chunks with every state kept (full fidelity)
        dict(name="trajectory_full", kind="trajectory", B=16, L=512, D=2048, N=16, io="bf16", st="f16", every=1,
             mu=-2.0, sigma=0.5),
        # the complex-A variant on a few contexts
        dict(name="complex_encode", kind="complex", B=8, L=3000, D=2048, N=16, io="bf16", out="bf16", st="f32",
             mu=-2.0, sigma=0.5),
        # 256 queries against the 10,000-chunk corpus and their 32-token
        # prefill from the retrieved states
        dict(name="query_path", kind="query", B=256, L=32, D=1024, N=16, M=10000, E=384, io="bf16", out="bf16",
             st="f16", prepared=True, mu=-2.0, sigma=0.5),
        # a handful of queries against a large index
        dict(name="retrieve_large", kind="topk", Q=16, M=100003, E=384, k=3, prepared=True),
        # joint episodic and corpus injection of whole 24-layer states
        dict(name="joint_inject", kind="fuse", Q=32, S=24 * 1024 * 16, ke=3, kc=3, k=3, Me=50, Mc=400, st="f16"),
        # one consolidation: 64 chunks routed and deposited
        dict(name="consolidate", kind="smc", C=64, E=384, ndom=5, nsub=4, S=24 * 4096, st="f16"),
    ]


def _log(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    kind = rng.choice(["step", "scan", "encode", "states", "long", "trajectory", "complex", "query", "topk", "fuse",
                       "smc"])
    io = rng.choice(["bf16", "bf16", "f32"])
    sc = dict(N=16, io=io, out=io, st=rng.choice(["f16", "f32"]), mu=-2.0, sigma=0.5)
    if kind == "step":  # a few tokens of running sessions
        return dict(sc, kind="scan", B=_log(rng, 1, 64), L=rng.randint(1, 9), D=8 * _log(rng, 16, 256), y=True, z=True,
                    h0=True)
    if kind == "scan":  # one short layer
        return dict(sc, kind="scan", B=_log(rng, 1, 8), L=_log(rng, 65, 2048), D=8 * _log(rng, 8, 128), y=True, z=True,
                    h0=rng.random() < 0.5)
    if kind == "encode":  # batches of documents, with outputs
        return dict(sc, kind="encode", B=_log(rng, 3, 64), L=_log(rng, 200, 3000), D=8 * _log(rng, 64, 256), y=True,
                    z=rng.random() < 0.7, h0=rng.random() < 0.5)
    if kind == "states":  # final states only, of 16, 32 or 64 a channel
        return dict(sc, kind="encode", B=_log(rng, 8, 96), L=_log(rng, 300, 3000), D=8 * _log(rng, 64, 192),
                    N=rng.choice([16, 32, 64]), y=False, z=False, h0=False, mu=-3.0, sigma=1.0)
    if kind == "long":
        return dict(sc, kind="encode", B=rng.randint(1, 2), L=_log(rng, 8000, 65536), D=8 * _log(rng, 96, 256), y=True,
                    z=True, h0=False)
    if kind == "trajectory":
        return dict(kind="trajectory", B=_log(rng, 2, 16), L=_log(rng, 100, 512), D=8 * _log(rng, 64, 256), N=16, io=io,
                    st=rng.choice(["f16", "f32"]), every=rng.choice([1, 2, 5, 8, 64]), mu=-2.0, sigma=0.5)
    if kind == "complex":
        return dict(sc, kind="complex", B=_log(rng, 1, 8), L=_log(rng, 200, 3000), D=8 * _log(rng, 64, 256))
    if kind == "query":
        return dict(sc, kind="query", B=_log(rng, 1, 256), L=rng.randint(8, 64), D=8 * _log(rng, 64, 128),
                    M=_log(rng, 500, 10000), E=rng.choice([128, 256, 384, 388, 768]), prepared=rng.random() < 0.7)
    if kind == "topk":
        return dict(kind="topk", Q=_log(rng, 1, 300), M=_log(rng, 500, 100003), E=rng.choice([128, 384, 388, 768]),
                    k=rng.choice([1, 3, 5, 10]), prepared=rng.random() < 0.6)
    if kind == "fuse":
        k = rng.choice([1, 3, 5])
        return dict(kind="fuse", Q=_log(rng, 1, 64), S=8 * _log(rng, 2048, 49152), ke=k, kc=k, k=k, Me=50, Mc=400,
                    st=rng.choice(["f16", "f32"]))
    return dict(kind="smc", C=_log(rng, 1, 300), E=rng.choice([128, 384, 768]), ndom=rng.randint(2, 8),
                nsub=rng.randint(2, 8), S=8 * _log(rng, 512, 12288), st=rng.choice(["f16", "f32"]))


# ---------------------------------------------------------------- inputs
def _gen(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    return g


def _normal(g, shape, dtype, std=1.0):
    out = torch.empty(shape, dtype=dtype, device=DEV)
    step = max(1, (1 << 26) // max(1, out[0].numel()))
    for i in range(0, shape[0], step):
        part = out[i:i + step]
        part.copy_(torch.randn(part.shape, generator=g, device=DEV) * std)
    return out


def _unit(v):
    return (v.double() / v.double().norm(dim=-1, keepdim=True)).float()


def _scan_inputs(c, g):
    B, L, D, N, t = c["B"], c["L"], c["D"], c["N"], _T[c["io"]]
    gate = c.get("z", c["kind"] in ("complex", "query"))
    read = c.get("y", c["kind"] in ("complex", "query"))
    d = dict(x=_normal(g, (B, L, D), t), A=torch.rand((D, N), generator=g, device=DEV) * 15 + 1,
             B=_normal(g, (B, L, N), t, N ** -0.5))
    dt = torch.empty((B, L, D), dtype=t, device=DEV)
    for b in range(B):
        v = torch.randn((L, D), generator=g, device=DEV) * c["sigma"] + c["mu"]
        dt[b] = torch.nn.functional.softplus(v).to(t)
    d["dt"] = dt
    d["C"] = _normal(g, (B, L, N), t, N ** -0.5) if read else None
    d["Dskip"] = torch.randn((D,), generator=g, device=DEV) if read else None
    d["z"] = _normal(g, (B, L, D), t) if gate else None
    d["h0"] = _normal(g, (B, D, N), _T[c["st"]]) if c.get("h0") else None
    if c["kind"] == "complex":  # the frequencies pi k of the diagonal
        d["A_im"] = (torch.arange(N, device=DEV, dtype=torch.float64) * math.pi).float().repeat(D, 1)
    return d


def _search_inputs(Q, M, E, g):
    keys = _unit(torch.randn((M, E), generator=g, device=DEV))
    q = torch.randn((Q, E), generator=g, device=DEV)
    near = Q // 2  # half of the queries ask for a stored chunk, half for none
    if near:
        rows = torch.randint(0, M, (near,), generator=g, device=DEV)
        q[:near] = keys[rows] + 0.05 * q[:near]
    return _unit(q), keys


def _inputs(c, seed):
    g = _gen(seed)
    if c["kind"] in ("scan", "encode", "trajectory", "complex"):
        return _scan_inputs(c, g)
    if c["kind"] == "query":
        d = _scan_inputs(c, g)
        d["query"], d["index"] = _search_inputs(c["B"], c["M"], c["E"], g)
        d["store"] = _normal(g, (c["M"], c["D"], c["N"]), _T[c["st"]])
        return d
    if c["kind"] == "topk":
        q, keys = _search_inputs(c["Q"], c["M"], c["E"], g)
        return dict(query=q, index=keys)
    if c["kind"] == "fuse":
        def cand(M, k):
            rows = torch.stack([torch.randperm(M, generator=g, device=DEV)[:k] for _ in range(c["Q"])]).int()
            score = torch.rand((c["Q"], k), generator=g, device=DEV, dtype=torch.float64).sort(
                dim=1, descending=True).values
            return rows, score
        d = dict(es=_normal(g, (c["Me"], c["S"]), _T[c["st"]]), cs=_normal(g, (c["Mc"], c["S"]), _T[c["st"]]),
                 sem=_normal(g, (20, c["S"]), _T[c["st"]]))
        d["ei"], d["ew"] = cand(c["Me"], c["ke"])
        d["ci"], d["cw"] = cand(c["Mc"], c["kc"])
        d["row"] = torch.randint(0, 20, (c["Q"],), generator=g, device=DEV).int()
        return d
    E, nd, ns = c["E"], c["ndom"], c["nsub"]
    dom = _unit(torch.randn((nd, E), generator=g, device=DEV))
    sub = _unit(dom[:, None] + 0.3 * torch.randn((nd, ns, E), generator=g, device=DEV) / math.sqrt(E))
    at = torch.randint(0, nd * ns, (c["C"],), generator=g, device=DEV)
    emb = _unit(sub.reshape(-1, E)[at] + 0.05 * torch.randn((c["C"], E), generator=g, device=DEV) / math.sqrt(E))
    return dict(emb=emb, dom=dom, sub=sub, at=at, states=_normal(g, (nd * ns, c["S"]), _T[c["st"]]),
                contrib=_normal(g, (c["C"], c["S"]), _T[c["st"]]))


def prepare(case, seed):
    c = case
    s = dict(_inputs(c, seed), c=c)
    if c["kind"] == "scan":  # a serving loop keeps its buffers and descriptor
        s["desc"] = P.scan_desc(c["B"], c["L"], c["D"], c["N"], P._DT[_T[c["io"]]], P._DT[_T[c["out"]]],
                                P._DT[_T[c["st"]]])
        s["bytes"] = P.scan_workspace_bytes(s["desc"])
        s["ws"] = torch.empty(s["bytes"], dtype=torch.uint8, device=DEV) if s["bytes"] else None
        s["yout"] = torch.empty((c["B"], c["L"], c["D"]), dtype=_T[c["out"]], device=DEV)
        s["hT"] = torch.empty((c["B"], c["D"], c["N"]), dtype=_T[c["st"]], device=DEV)
    elif c["kind"] in ("query", "topk") and c["prepared"]:  # the index is embedded offline
        s["prep"] = P.prepare_index(s["index"])
    elif c["kind"] == "fuse":
        s["h0out"] = torch.empty((c["Q"], c["S"]), dtype=_T[c["st"]], device=DEV)
    return s


def run(s):
    c = s["c"]
    kind = c["kind"]
    if kind == "scan":
        P.scan_encode(s["desc"], s["x"], s["dt"], s["A"], s["B"], s["C"], s["z"], s["Dskip"], s["h0"], s["yout"],
                      s["hT"], s["ws"], s["bytes"])
        return s["yout"], s["hT"]
    if kind == "encode":
        y, h = P.scan(s["x"], s["dt"], s["A"], s["B"], s["C"], s["z"], s["Dskip"], s["h0"], out_dtype=_T[c["out"]],
                      state_dtype=_T[c["st"]], want_y=c["y"])
        return (y, h) if c["y"] else h
    if kind == "trajectory":
        return P.trajectory(s["x"], s["dt"], s["A"], s["B"], c["every"], state_dtype=_T[c["st"]])[0]
    if kind == "complex":
        return P.scan_complex(s["x"], s["dt"], s["A"], s["A_im"], s["B"], s["C"], s["z"], s["Dskip"],
                              out_dtype=_T[c["out"]], state_dtype=_T[c["st"]])
    if kind == "query":
        return P.query_prefill(s["query"], s["index"], s["store"], s["x"], s["dt"], s["A"], s["B"], s["C"], s["z"],
                               s["Dskip"], prepared=s.get("prep"), out_dtype=_T[c["out"]])
    if kind == "topk":
        if c["prepared"]:
            return P.topk_prepared(s["query"], s["index"], s["prep"], c["k"])
        return P.topk(s["query"], s["index"], c["k"])
    if kind == "fuse":
        P.inject_fuse(s["es"], s["ei"], s["ew"], s["cs"], s["ci"], s["cw"], c["k"], 0.1, s["h0out"], s["sem"], s["row"],
                      0.5)
        return s["h0out"]
    dom, sub, flat = P.route(s["emb"], s["dom"], s["sub"])
    P.smc_consolidate(s["states"], s["contrib"], flat, 0.25)
    return dom, sub, s["states"]


# ------------------------------------------------------------------ work
def work(case):
    """Inputs read once, outputs written once.  Operations of a scan per
    (token, channel, state): the decay's product and exponential, its
    product with B, the state's and the readout's multiply-add; per (token,
    channel): dt x, skip and gate."""
    c = case
    kind = c["kind"]
    if kind in ("scan", "encode", "trajectory", "complex", "query"):
        B, L, D, N, i, st = c["B"], c["L"], c["D"], c["N"], _SIZE[c["io"]], _SIZE[c["st"]]
        read = c.get("y", kind != "trajectory")
        gate = c.get("z", kind in ("complex", "query"))
        pair = 2 if kind == "complex" else 1
        n = B * L * D * (2 + gate) * i + B * L * N * (1 + read) * i + D * N * 4 * pair
        n += read * (B * L * D * _SIZE[c.get("out", c["io"])] + D * 4)
        flops = B * L * D * (N * ((15 if kind == "complex" else 5) + 2 * read) + 1 + 8 * gate + 2 * read)
        if kind == "trajectory":
            n += B * (L // c["every"]) * D * N * st
        else:
            n += B * D * N * st * pair * (2 if c.get("h0") or kind == "query" else 1)
        if kind == "query":
            n += c["M"] * c["E"] * (2 if c["prepared"] else 4) + B * c["E"] * 4 + B * 4
            flops += 2 * B * c["M"] * c["E"]
        return dict(bytes=n, flops=flops)
    if kind == "topk":
        return dict(bytes=c["M"] * c["E"] * (2 if c["prepared"] else 4) + c["Q"] * c["E"] * 4 + c["Q"] * c["k"] * 12,
                    flops=2 * c["Q"] * c["M"] * c["E"])
    if kind == "fuse":
        return dict(bytes=c["Q"] * ((c["k"] + 2) * c["S"] * _SIZE[c["st"]] + (c["ke"] + c["kc"]) * 12),
                    flops=c["Q"] * c["S"] * 2 * (c["k"] + 1))
    R, st = c["ndom"] * c["nsub"], _SIZE[c["st"]]
    return dict(bytes=(2 * min(R, c["C"]) + c["C"]) * c["S"] * st + 4 * c["E"] * (c["C"] + c["ndom"] + R),
                flops=3 * c["C"] * c["S"] + 2 * c["C"] * c["E"] * (c["ndom"] + c["nsub"]))


def tolerance(case):
    c = case
    if c["kind"] == "topk":  # exact by contract: fp64 sums in feature order
        return "exact"
    if c["kind"] in ("fuse", "smc"):  # 32-bit sums, stored in the state type
        return dict(rel=1.2e-3 if c["st"] == "f16" else 5e-7, max=5e-3 if c["st"] == "f16" else 1e-5)
    if c.get("out", c["io"]) == "bf16" and c["kind"] != "trajectory" and c.get("y", True):
        return dict(rel=7e-3, max=2e-2)  # bf16 outputs: 1.7e-3 off by their rounding alone
    if c["st"] == "f16":
        return dict(rel=8e-4, max=4e-3)  # fp16 states: 2e-4 off by their rounding alone
    # everything in 32 bits: 7e-8 off, 3e-7 with the complex A's sines
    return dict(rel=1.2e-6 if c["kind"] == "complex" else 4e-7, max=5e-5)


# ----------------------------------------------------------------- exact
def _exact_scan(c, d, h0=None):
    B, L, D, N = c["B"], c["L"], c["D"], c["N"]
    read = d["C"] is not None
    A = d["A"].double()
    if c["kind"] == "complex":
        A = torch.complex(A, d["A_im"].double())
    h = torch.zeros((B, D, N), dtype=A.dtype, device=DEV) if h0 is None else h0.to(A.dtype)
    every = c.get("every", 0) if c["kind"] == "trajectory" else 0
    y = torch.empty((B, L, D), dtype=torch.float64, device=DEV) if read else None
    traj = torch.empty((B, L // every, D, N), dtype=torch.float64, device=DEV) if every else None
    for t in range(L):
        dt = d["dt"][:, t].double()
        x = d["x"][:, t].double()
        h = torch.exp(-dt[:, :, None] * A) * h
        h += (dt * x)[:, :, None] * d["B"][:, t].double()[:, None, :]
        if read:
            v = torch.matmul(h.real if h.is_complex() else h, d["C"][:, t].double()[:, :, None])[:, :, 0]
            v = v + d["Dskip"].double() * x
            if d["z"] is not None:
                z = d["z"][:, t].double()
                v = v * z * torch.sigmoid(z)
            y[:, t] = v
        if every and (t + 1) % every == 0:
            traj[:, (t + 1) // every - 1] = h
    if every:
        return traj
    hT = torch.view_as_real(h) if h.is_complex() else h
    return (y, hT) if read else hT


def exact(case, seed):
    c = case
    d = _inputs(c, seed)
    if c["kind"] in ("scan", "encode", "trajectory", "complex"):
        return _exact_scan(c, d, d["h0"])
    if c["kind"] == "query":
        at = torch.matmul(d["query"].double(), d["index"].double().t().contiguous()).argmax(dim=1)
        y, h = _exact_scan(c, d, d["store"][at])
        return None, y, h
    if c["kind"] == "topk":
        s = torch.matmul(d["query"].double(), d["index"].double().t().contiguous())
        return None, s.topk(c["k"], dim=1).values
    if c["kind"] == "fuse":
        score = torch.cat([d["ew"], d["cw"]], dim=1)
        top = score.topk(c["k"], dim=1)
        w = torch.softmax(top.values / 0.1, dim=1)
        out = torch.empty((c["Q"], c["S"]), dtype=torch.float64, device=DEV)
        for q in range(c["Q"]):
            rows = torch.cat([d["es"][d["ei"][q].long()], d["cs"][d["ci"][q].long()]])[top.indices[q]].double()
            out[q] = (w[q][:, None] * rows).sum(dim=0) + 0.5 * d["sem"][d["row"][q].long()].double()
        return out
    s = d["states"].double()
    flat = d["at"].tolist()  # each chunk lies next to its own sub-cluster
    for i, r in enumerate(flat):
        s[r] = 0.75 * s[r] + 0.25 * d["contrib"][i].double()
    return None, None, s
