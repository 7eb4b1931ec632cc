"""Performance cases of the WaveFilter filter+attend path.

A case is one call that a decoder of a diffusion language model makes for one
layer of one denoising step (or, for "staged" and "dwt", the staged calls and
the one-time transform of the prompt keys).  Sizes follow the workloads of
synth.WORKLOADS and bench.py; inputs follow the recipe of synth (AR(1) keys
with planted 16-token needles, queries leaning towards them), drawn on the
GPU.  Every case runs with buffers that a serving loop keeps (workspace,
outputs), except the grouped and transform calls, whose entry points allocate
their own.

The selected indices are not returned: one pair of near-equal scores in the
other order moves all positions between the two in an ascending list.  The
attention output depends on every selected token, and the staged case
returns the scores themselves.
"""
from __future__ import annotations

import math

import torch

import paper_2606_00724_amd as wf

_NEEDLE = 16


def listed():
    return [
        # the smallest call: two fp32 heads, a 1K prompt; launches and latency
        _case("fused", "tiny_f32", batch=1, heads=2, L=1024, d=64, B=32, dtype="f32",
              rho=0.95, needles=1, J=3, k=128),
        # one layer of an 8B model at a 4K prompt, bf16
        _case("fused", "layer8b", batch=1, heads=32, L=4096, d=128, B=32, rho=0.95,
              needles=4, J=3, k=512),
        # the same layer with fp32 keys (accuracy studies, fp32 models)
        _case("fused", "layer8b_f32", batch=1, heads=32, L=4096, d=128, B=32, dtype="f32",
              rho=0.95, needles=4, J=3, k=512),
        # long-context serving, one of 32 layers
        _case("fused", "long16k", batch=1, heads=32, L=16384, d=128, B=32, needles=8, J=4,
              k=1024),
        # the headline workload: a batch of four 32K prompts
        _case("fused", "headline32k", batch=4, heads=32, L=32768, d=128, B=64, needles=8, J=5,
              k=2048),
        # 128K prompt with the smoother wavelet
        _case("fused", "stress128k_db2", batch=1, heads=32, L=131072, d=128, B=32, rho=0.99,
              needles=16, wavelet="db2", J=6, k=4096),
        # every denoising step after the first: the prompt's A_J is kept
        _case("cached", "cached32k", batch=4, heads=32, L=32768, d=128, B=64, needles=8, J=5,
              k=2048),
        # the paper's own two-scale schedule
        _case("recursive", "recursion32k", batch=4, heads=32, L=32768, d=128, B=64, needles=8,
              J=2, k=2048, m1=0.5, m2=0.25),
        # one selection for all heads of a sequence; a prompt length that is
        # no multiple of 2^J, a generation tail and an odd query block
        _case("shared", "shared8k_ragged", batch=2, heads=32, L=8211, d=128, B=45, G=64,
              needles=6, J=4, k=1024),
        # grouped-query attention: 8 KV heads, 4 query heads each (128 rows)
        _case("grouped", "grouped16k", batch=2, heads=8, L=16384, d=128, B=32, group=4,
              needles=8, J=4, k=1024),
        # the staged calls one by one, as a program does that keeps the
        # coefficients, scores and the sparse cache
        _case("staged", "staged8b", batch=1, heads=32, L=4100, d=128, B=32, G=32, rho=0.95,
              needles=4, J=3, k=512),
        # the transform that a cached 128K prompt pays once (the staged case
        # has the Haar one)
        _case("dwt", "dwt128k_db2", batch=1, heads=32, L=131072, d=128, B=32, rho=0.99,
              needles=16, wavelet="db2", J=6, k=4096),
    ]


def _case(kind, name, *, batch, heads, L, d, B, J, k, dtype="bf16", rho=0.98, needles=4,
          wavelet="haar", boundary="symmetric", G=0, group=1, m1=0.0, m2=0.0, m3=0.0):
    S = min(L >> J, -(-2 * k // (1 << J)))  # a pool of twice the budget
    c = dict(kind=kind, batch=batch, heads=heads, L=L, d=d, B=B, J=J, S=S, k=k, dtype=dtype,
             rho=rho, needles=needles, wavelet=wavelet, boundary=boundary, G=G, group=group,
             m1=m1, m2=m2, m3=m3)
    if name is not None:
        c["name"] = name
    return c


def draw(rng):
    kind = rng.choice(["fused", "fused", "fused", "cached", "recursive", "shared", "grouped",
                       "staged", "dwt"])
    dtype = "f32" if kind in ("fused", "cached", "staged", "dwt") and rng.random() < 0.2 else "bf16"
    d = rng.choice([64, 128, 128, 128])
    units = int(round(2 ** rng.uniform(1, 7)))  # 2 .. 128
    batch = rng.choice([b for b in (1, 2, 3, 4) if b <= units])
    heads = max(1, units // batch)
    # at most the headline's keys, an eighth of it where fp32 arithmetic or
    # more query rows make a key dearer
    most = (1 << 29) >> (3 if dtype == "f32" or kind in ("grouped", "staged") else 0)
    top = min(131072, most // (batch * heads * d))
    L = int(round(2 ** rng.uniform(10, math.log2(max(2048, top)))))
    if rng.random() < 0.6:
        L -= L % 64
    B = rng.choice([8, 16, 17, 32, 32, 32, 45, 48, 64, 64])
    group = 1
    if kind == "grouped":
        group = rng.choice([2, 4, 4, 8])
        B = min(B, 256 // group)
    wavelet = "db2" if kind != "recursive" and rng.random() < 0.25 else "haar"
    boundary = rng.choice(["symmetric", "symmetric", "periodic"])
    # about 512 to 2048 coefficients, as the workloads have
    J = max(2, min(6, int(math.log2(L)) - rng.choice([9, 9, 10, 11])))
    if kind == "recursive":
        J = rng.choice([2, 2, 3])
    ms = [rng.choice([0.25, 0.5]) for _ in range(3)]
    k = max(32, int(L / 2 ** rng.uniform(3, 5)))
    G = rng.choice([0, 0, 0, 32, 64, 33]) if kind != "dwt" else 0
    return _case(kind, None, batch=batch, heads=heads, L=L, d=d, B=B, J=J, k=k, dtype=dtype,
                 rho=rng.choice([0.95, 0.98, 0.99]), needles=rng.choice([1, 4, 8]),
                 wavelet=wavelet, boundary=boundary, G=G, group=group,
                 m1=ms[0] if kind == "recursive" else 0.0,
                 m2=ms[1] if kind == "recursive" else 0.0,
                 m3=ms[2] if kind == "recursive" and J == 3 else 0.0)


# ------------------------------------------------------------ inputs

def _inputs(c, seed):
    """Q, K, V, Kg, Vg on the GPU, from the seed alone."""
    dev = torch.device("cuda")
    gen = torch.Generator(device=dev)
    gen.manual_seed(1000003 * int(seed) + 17)
    b, h, L, d, B, G = c["batch"], c["heads"], c["L"], c["d"], c["B"], c["G"]
    rows = B * c["group"]
    dt = torch.bfloat16 if c["dtype"] == "bf16" else torch.float32

    def normal(*shape):
        return torch.randn(shape, generator=gen, device=dev)

    u = normal(b, h, 1, d)
    u /= u.norm(dim=-1, keepdim=True)
    starts = torch.randint(0, L // _NEEDLE - 1, (b, c["needles"]), generator=gen, device=dev)
    rho = c["rho"]
    K = torch.empty((b, h, L, d), dtype=dt, device=dev)
    V = torch.empty_like(K)
    for i in range(b):
        x = normal(h, L, d)
        x[:, 1:] *= math.sqrt(1 - rho * rho)
        s = 1
        while s < L and rho ** s > 1e-6:  # AR(1) by doubling
            x[:, s:] += rho ** s * x[:, :-s].clone()
            s *= 2
        x += 0.3 * normal(h, L, d)
        at = (starts[i, :, None] * _NEEDLE + torch.arange(_NEEDLE, device=dev)).reshape(-1).unique()
        x[:, at] += 3.0 * u[i]
        K[i] = x
        V[i] = normal(h, L, d)
    Q = (normal(b, h, rows, d) / math.sqrt(d) + 2.0 * u).to(dt)
    if c["kind"] == "grouped":  # a KV head's query heads are adjacent
        Q = Q.reshape(b, h * c["group"], B, d)
    Kg = normal(b, h, G, d).to(dt) if G else None
    Vg = normal(b, h, G, d).to(dt) if G else None
    return Q, K, V, Kg, Vg


def _params(c):
    return wf.make_params(batch=c["batch"], heads=c["heads"], ctx_len=c["L"], head_dim=c["d"],
                          q_len=c["B"] * c["group"], levels=c["J"], segments=c["S"],
                          budget=c["k"], gen_len=c["G"], wavelet=c["wavelet"],
                          boundary=c["boundary"], dtype=c["dtype"])


def _props(c):
    return [c["m1"], c["m2"], c["m3"]][:c["J"]]


def prepare(case, seed):
    c = case
    wf.wf_init()
    p = _params(c)
    Q, K, V, Kg, Vg = _inputs(c, seed)
    dev = Q.device
    st = dict(case=c, p=p, Q=Q, K=K, V=V, Kg=Kg, Vg=Vg)
    kind = c["kind"]
    if kind == "dwt":
        return dict(case=c, p=p, K=K)
    st["O"] = torch.empty_like(Q)
    if kind == "fused":
        st["ws"] = wf.alloc_workspace(p, wf.OP_FUSED, dev)
    elif kind == "cached":
        st["approx"] = wf.dwt_approx(p, K)
        st["ws"] = wf.alloc_workspace(p, wf.OP_CACHED, dev)
    elif kind == "shared":
        st["ws"] = wf.alloc_workspace(p, wf.OP_SHARED, dev)
    elif kind == "recursive":
        nb = wf.recursive_workspace_bytes(p, _props(c))
        st["ws"] = torch.empty(nb, dtype=torch.uint8, device=dev)
        st["tok"] = torch.empty((c["batch"], c["heads"], 2 * wf.recursion_counts(p, _props(c))[0]),
                                dtype=torch.int32, device=dev)
    elif kind == "staged":
        b, h, d = c["batch"], c["heads"], c["d"]
        keff = wf.effective_budget(p)
        rows = keff + c["L"] % (1 << c["J"]) + c["G"]

        def new(*shape, dtype):
            return torch.empty((b, h) + shape, dtype=dtype, device=dev)

        st.update(
            approx=new(c["L"] >> c["J"], d, dtype=torch.float32),
            W=new(c["L"] >> c["J"], dtype=torch.float32),
            seg=new(c["S"], dtype=torch.int32), tok=new(keff, dtype=torch.int32),
            Ks=new(rows, d, dtype=K.dtype), Vs=new(rows, d, dtype=K.dtype), rows=rows,
            ws_skim=wf.alloc_workspace(p, wf.OP_SKIM, dev),
            ws_scan=wf.alloc_workspace(p, wf.OP_SCAN, dev),
            ws_attn=wf.alloc_workspace(p, wf.OP_ATTN, dev))
    return st


def run(state):
    s, p, kind = state, state["p"], state["case"]["kind"]
    if kind == "dwt":
        return wf.dwt_approx(p, s["K"])
    Q, K, V, Kg, Vg, O = s["Q"], s["K"], s["V"], s["Kg"], s["Vg"], s["O"]
    if kind == "fused":
        wf.wf_filter_attend(p, Q, K, V, Kg, Vg, O, None, None, s["ws"])
    elif kind == "cached":
        wf.wf_filter_attend_cached(p, Q, s["approx"], K, V, Kg, Vg, O, None, None, s["ws"])
    elif kind == "shared":
        wf.wf_filter_attend_shared(p, Q, K, V, Kg, Vg, O, None, None, s["ws"])
    elif kind == "recursive":
        wf.wf_filter_attend_recursive(p, _props(s["case"]), Q, K, V, Kg, Vg, O, s["tok"], s["ws"])
    elif kind == "grouped":
        return wf.filter_attend_grouped(p, s["case"]["group"], Q, K, V, Kg, Vg)
    else:
        wf.wf_dwt_keys(p, K, s["approx"])
        wf.wf_skim_score(p, Q, s["approx"], s["W"], s["seg"], s["ws_skim"])
        wf.wf_scan_select(p, Q, K, s["seg"], None, s["tok"], s["ws_scan"])
        wf.wf_gather_kv(p, K, V, s["tok"], Kg, Vg, s["Ks"], s["Vs"])
        wf.wf_sparse_attn(p, Q, s["Ks"], s["Vs"], s["rows"], O, s["ws_attn"])
        return {"approx": s["approx"], "W": s["W"], "O": O}
    return O


# ------------------------------------------------------------ work

def _counts(c):
    """Rows a unit's attention reads, and the recursion's candidates."""
    nJ = c["L"] >> c["J"]
    if c["kind"] != "recursive":
        return min(c["k"], c["S"] << c["J"]), []
    n, cand = nJ, []
    for m in reversed(_props(c)):
        cand.append(n)
        keep = max(1, min(n, math.ceil(m * n)))
        n = 2 * keep
    return 2 * keep, cand


def work(case):
    c = case
    U, L, d, J = c["batch"] * c["heads"], c["L"], c["d"], c["J"]
    e = 2 if c["dtype"] == "bf16" else 4
    rows, R, G = c["B"] * c["group"], c["L"] % (1 << c["J"]), c["G"]
    nJ, pool = L >> J, c["S"] << J
    dwt_flops = 2 * (2 if c["wavelet"] == "haar" else 4) * (L - R) * d
    if c["kind"] == "dwt":
        return {"bytes": U * d * (L * e + nJ * 4), "flops": U * dwt_flops}
    keep, cand = _counts(c)
    kv = keep + R + G
    # the values of the kept rows, the tail, queries in and outputs out; the
    # keys once (the kept rows' keys are among them)
    by = kv * d * e + G * d * e + 2 * rows * d * e
    fl = 4 * rows * kv * d
    if c["kind"] == "cached":
        by += nJ * d * 4 + pool * d * e  # A_J and the pool's keys
        fl += 2 * rows * (nJ + pool) * d
    elif c["kind"] == "recursive":
        by += L * d * e
        fl += dwt_flops + 2 * rows * sum(cand) * d
    else:
        by += L * d * e
        fl += dwt_flops + 2 * rows * (nJ + pool) * d
        if c["kind"] == "staged":
            # A_J, W and the sparse cache are outputs, and inputs of the next call
            by += 2 * nJ * d * 4 + nJ * 4 + 2 * 2 * kv * d * e
    return {"bytes": U * by, "flops": U * fl}


def tolerance(case):
    # about four times the measured distance from a 64-bit evaluation: 2.3e-3
    # where the output and the probabilities round to bf16, 2e-7 for fp32
    # attention, 6e-8 (Haar 3e-8) for the transform
    if case["kind"] == "dwt":
        return {"rel": 3e-7}
    return {"rel": 1e-2} if case["dtype"] == "bf16" else {"rel": 1e-6}


# ------------------------------------------------------------ 64-bit evaluation

_R3 = math.sqrt(3.0)
_DB2 = [(1 + _R3) / (4 * math.sqrt(2)), (3 + _R3) / (4 * math.sqrt(2)),
        (3 - _R3) / (4 * math.sqrt(2)), (1 - _R3) / (4 * math.sqrt(2))]


def _dwt(x, c, levels):
    """[n, d] -> [n >> levels, d], n a multiple of 2^levels."""
    for _ in range(levels):
        n = x.shape[0]
        if c["wavelet"] == "haar":
            x = (x[0::2] + x[1::2]) / math.sqrt(2.0)
            continue
        ext = [n - 1, n - 2] if c["boundary"] == "symmetric" else [0, 1 % n]
        y = torch.cat([x, x[ext]])
        x = sum(_DB2[m] * y[m:m + n:2] for m in range(4))
    return x


def _weights(Q, A, scale):
    return torch.softmax((Q @ A.T) * scale, dim=-1).sum(0)


def _top(w, k):
    return torch.sort(w, descending=True, stable=True).indices[:k].sort().values


def exact(case, seed):
    c = case
    U, L, d, J = c["batch"] * c["heads"], c["L"], c["d"], c["J"]
    rows = c["B"] * c["group"]
    Q, K, V, Kg, Vg = _inputs(c, seed)
    qshape = Q.shape
    Q, K, V = Q.reshape(U, rows, d), K.reshape(U, L, d), V.reshape(U, L, d)
    Lf, nJ, S = (L >> J) << J, L >> J, c["S"]
    scale = 1.0 / math.sqrt(d)
    dev = Q.device
    rest = torch.arange(Lf, L, device=dev)
    keep = min(c["k"], S << J)
    if c["kind"] == "dwt":
        A = torch.stack([_dwt(K[u, :Lf].double(), c, J) for u in range(U)])
        return A.reshape(c["batch"], c["heads"], nJ, d)

    def pool_of(seg):
        return (seg[:, None] * (1 << J) + torch.arange(1 << J, device=dev)).reshape(-1)

    toks, As, Ws = [], [], []
    if c["kind"] == "recursive":
        for u in range(U):
            q, k, mu = Q[u].double(), K[u].double(), torch.arange(Lf, device=dev)
            for b, m in zip(range(J, 0, -1), reversed(_props(c))):
                A = _dwt(k[mu], c, b)
                n = A.shape[0]
                cb = max(1, min(n, math.ceil(float(torch.tensor(m, dtype=torch.float32)) * n)))
                kept = _top(_weights(q, A, scale), cb)
                mu = mu[(kept[:, None] * (1 << b) + torch.arange(1 << b, device=dev)).reshape(-1)]
            toks.append(mu)
    elif c["kind"] == "shared":
        h = c["heads"]
        for b in range(c["batch"]):
            us = range(b * h, (b + 1) * h)
            W = sum(_weights(Q[u].double(), _dwt(K[u, :Lf].double(), c, J), scale) for u in us)
            pool = pool_of(_top(W, S))
            W2 = sum(_weights(Q[u].double(), K[u, pool].double(), scale) for u in us)
            toks += [pool[_top(W2, keep)]] * h
    else:
        for u in range(U):
            q = Q[u].double()
            A = _dwt(K[u, :Lf].double(), c, J)
            W = _weights(q, A, scale)
            pool = pool_of(_top(W, S))
            toks.append(pool[_top(_weights(q, K[u, pool].double(), scale), keep)])
            if c["kind"] == "staged":
                As.append(A)
                Ws.append(W)
    O = torch.empty((U, rows, d), dtype=torch.float64, device=dev)
    for u in range(U):
        at = torch.cat([toks[u], rest])
        k, v = K[u, at].double(), V[u, at].double()
        if c["G"]:
            k = torch.cat([k, Kg.reshape(U, -1, d)[u].double()])
            v = torch.cat([v, Vg.reshape(U, -1, d)[u].double()])
        O[u] = torch.softmax((Q[u].double() @ k.T) * scale, dim=-1) @ v
    O = O.reshape(qshape)
    if c["kind"] == "staged":
        return {"approx": torch.stack(As).reshape(c["batch"], c["heads"], nJ, d),
                "W": torch.stack(Ws).reshape(c["batch"], c["heads"], nJ), "O": O}
    return O
