"""The calls that a user of this library makes, as cases to be timed and compared.

A case is one call (or the two calls of a backward) through the public entry points on the shapes
of this repository's own workloads: the 20M-slot decode layer from one token to 1024, the 1M-slot
prefill layer, the Tucker layer with implicit value expansion and its projection, one memory layer
of the paper's UltraMem-1.6B-x12 model, the query front-end, and the backward of the three layers
that train.  ``draw`` gives further cases of the same ranges: odd token counts and key counts, other
widths, both value types, raw and SoftMax weights, with and without expansion and several cores.

Inputs are made on the GPU from the seed alone (torch generators).  ``exact`` is the same
arithmetic in float64 with plain torch.
"""
from __future__ import annotations

import math

import torch

import paper_2411_12364_amd as U

DEV = "cuda"

LAYER = dict(op="forward", T=1, heads=2, dk=128, n_keys=1024, topk=32, topm=32, dv=512, bf16=True,
             softmax=False, rank=0, cores=1, expand=1, dv_virt=0, d_out=0, clusters=0)


def _layer(**kw):
    return {**LAYER, **kw}


DECODE = dict(n_keys=4480, dv=512)                                   # 20.07M slots of 1 KiB
PREFILL = dict(n_keys=1024, dv=1024)                                 # 1M slots of 2 KiB
TUCKER = dict(heads=4, n_keys=2048, topk=64, topm=64, dv=512, rank=2, expand=4, dv_virt=512,
              d_out=2048, clusters=8)                                # 4.2M virtual slots on 1M rows
ULTRAMEM = dict(heads=2, dk=448, n_keys=1792, topk=42, topm=42, dv=4096, rank=2, cores=2, expand=4,
                dv_virt=1024, d_out=2048)                            # one layer of UltraMem-1.6B-x12


def listed():
    return [
        # one sequence being decoded: the smallest call there is
        _layer(name="decode-20M-T1", T=1, **DECODE),
        # the decode batch of the headline benchmark
        _layer(name="decode-20M-T32", T=32, **DECODE),
        # the largest decode batch of the benchmark's sweep
        _layer(name="decode-20M-T1024", T=1024, **DECODE),
        # a prompt's tokens
        _layer(name="prefill-1M-T2048", T=2048, **PREFILL),
        # the same on tokens that cluster (rows repeat), Tucker scores, expansion, projection
        _layer(name="tucker-ive-4M-T4096", T=4096, **TUCKER),
        # the decode batch that the paper times inference with
        _layer(name="ultramem-1.6B-T512", T=512, **ULTRAMEM),
        # a small fp32 layer with SoftMax weights, three heads and sizes that divide nothing
        _layer(name="odd-softmax-f32-T333", T=333, heads=3, dk=96, n_keys=1001, topk=20, topm=24,
               dv=256, bf16=False, softmax=True),
        # the query front-end of the UltraMem layer: one new token per sequence ...
        dict(name="query-512x1", op="query", B=512, L=1, d_model=2048, conv_k=4, heads=2, dk=448,
             shared=True, history=True),
        # ... and prompts of a ragged length, with separate row and column queries
        dict(name="query-4x509", op="query", B=4, L=509, d_model=2048, conv_k=4, heads=2, dk=128,
             shared=False, history=False),
        # a training step's backward through pooling and scoring, value gradients by distinct row
        _layer(name="backward-prefill-1M", op="backward", T=2048, dense=False, **PREFILL),
        _layer(name="backward-tucker-4M", op="backward", T=4096, dense=False, **TUCKER),
        _layer(name="backward-ultramem-1.6B", op="backward", T=512, dense=False, **ULTRAMEM),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case of the ranges above; none costs more than the largest of them."""
    kind = rng.choice(["additive", "additive", "tucker", "ultramem", "query", "backward", "backward"])
    if kind == "query":
        L = _log(rng, 1, 600)
        return dict(op="query", B=max(1, min(512, 2048 // L) - rng.randrange(3)), L=L,
                    d_model=rng.choice([1024, 1536, 2048]), conv_k=rng.choice([3, 4]),
                    heads=rng.choice([1, 2, 4]), dk=rng.choice([64, 128, 256, 448]),
                    shared=rng.random() < 0.5, history=rng.random() < 0.5)
    op = "forward"
    if kind == "backward":
        op = "backward"
        kind = rng.choice(["additive", "tucker", "ultramem"])
    if kind == "additive":
        T = _log(rng, 1 if op == "forward" else 64, 2048)
        heads = rng.choice([1, 2, 2, 3])
        topk = rng.randint(8, 32)
        c = _layer(op=op, T=T, heads=heads, dk=rng.choice([64, 96, 128, 256]),
                   n_keys=_log(rng, 500, 4480 if T <= 1024 else 1800), topk=topk,
                   topm=rng.randint(8, 32), softmax=rng.random() < 0.3)
        c["bf16"] = rng.random() < 0.75
        c["dv"] = rng.choice([256, 512, 1024] if c["bf16"] else [128, 256, 512])
        if op == "forward" and rng.random() < 0.25:
            c["d_out"] = rng.choice([512, 1000])
    elif kind == "tucker":
        topk = rng.randint(16, 64)
        E = rng.choice([1, 4, 4])
        c = _layer(op=op, T=_log(rng, 64, 4096), heads=rng.choice([2, 4]), dk=128,
                   n_keys=2 * _log(rng, 256, 1024), topk=topk, topm=rng.randint(16, 64), dv=512,
                   rank=2, cores=rng.choice([1, 1, 2]), expand=E, dv_virt=512 if E > 1 else 0,
                   d_out=2048, clusters=rng.choice([0, 8]))
    else:
        c = _layer(op=op, **{**ULTRAMEM, "T": _log(rng, 32, 512), "topm": rng.randint(24, 42),
                             "cores": rng.choice([1, 2]), "dv": rng.choice([2048, 4096])})
    if op == "backward":
        # the dense gradient table where a program would hold (and clear) one; else by distinct row
        c["dense"] = c["n_keys"] ** 2 // c["expand"] * c["dv"] <= 1 << 27 and rng.random() < 0.5
    return c


# ---------------------------------------------------------------------------- inputs

def _gen(seed):
    return torch.Generator(device=DEV).manual_seed(int(seed))


def _randn(g, shape, std, dtype=torch.float32):
    return torch.empty(shape, dtype=dtype, device=DEV).normal_(0.0, std, generator=g)


def _cores(c):
    return max(1, c["cores"])


def _bag(c):
    return c["heads"] * c["topm"]


def _n_values(c):
    return c["n_keys"] ** 2 // c["expand"]


def _desc(c):
    d = U.umem_desc()
    d.heads, d.dk, d.n_keys, d.rank = c["heads"], c["dk"], c["n_keys"], max(1, c["rank"])
    d.topk, d.topm = c["topk"], c["topm"]
    d.grid = U.UMEM_GRID_TUCKER if c["rank"] else U.UMEM_GRID_ADD
    d.weight = U.UMEM_W_SOFTMAX if c["softmax"] else U.UMEM_W_RAW
    d.n_values, d.dv, d.expand = _n_values(c), c["dv"], c["expand"]
    d.vdtype = U.UMEM_BF16 if c["bf16"] else U.UMEM_F32
    d.dv_virt, d.d_out, d.cores = c["dv_virt"], c["d_out"], c["cores"]
    return d


def _queries(c, g):
    """[T, H, dk]: unit-variance queries over sqrt(dk), or tokens around a few centres."""
    shape, std = (c["T"], c["heads"], c["dk"]), 1.0 / math.sqrt(c["dk"])
    if not c["clusters"]:
        return _randn(g, shape, std), _randn(g, shape, std)
    z = torch.randint(0, c["clusters"], (c["T"],), generator=g, device=DEV)
    out = []
    for _ in range(2):
        centres = _randn(g, (c["clusters"],) + shape[1:], std)
        out.append(centres[z] + 0.1 * _randn(g, shape, std))
    return out[0].contiguous(), out[1].contiguous()


def _layer_inputs(c, seed):
    g = _gen(seed)
    H, n, dk, dv = c["heads"], c["n_keys"], c["dk"], c["dv"]
    s = {"q_row": None, "q_col": None}
    s["q_row"], s["q_col"] = _queries(c, g)
    s["k_row"] = _randn(g, (H, n, dk), 1.0 / math.sqrt(dk))
    s["k_col"] = _randn(g, (H, n, dk), 1.0 / math.sqrt(dk))
    r, h = c["rank"], _cores(c)
    s["core"] = _randn(g, (H, h, r, r) if h > 1 else (H, r, r), 1.0) if r else None
    s["values"] = _randn(g, (_n_values(c), dv), 1.0 / math.sqrt(dv),
                         torch.bfloat16 if c["bf16"] else torch.float32)
    s["perm"] = (torch.randperm(n * n, generator=g, device=DEV).to(torch.int32)
                 if c["expand"] > 1 else None)
    s["w_proj"] = s["w_out"] = None
    if c["op"] == "forward":
        k1 = c["expand"] * dv
        if c["dv_virt"]:
            s["w_proj"] = _randn(g, (c["dv_virt"], k1), 1.0 / math.sqrt(dv), torch.bfloat16)
        if c["d_out"]:
            k2 = c["dv_virt"] or dv
            s["w_out"] = _randn(g, (c["d_out"], k2), 1.0 / math.sqrt(k2), torch.bfloat16)
    else:
        # the gradient that comes back to the pooled rows
        s["d_pooled"] = _randn(g, (c["T"], c["expand"], dv), 1.0)
    return s


def _query_inputs(c, seed):
    g = _gen(seed)
    A, d = (1 if c["shared"] else 2), c["d_model"]
    return {
        "x": _randn(g, (c["B"], c["L"], d), 1.0),
        "hist": _randn(g, (c["B"], c["conv_k"] - 1, d), 1.0) if c["history"] else None,
        "conv_w": _randn(g, (c["conv_k"], d), 1.0 / math.sqrt(c["conv_k"])),
        "w_q": _randn(g, (A * c["heads"] * c["dk"], d), 1.0 / math.sqrt(d), torch.bfloat16),
        "gamma": 1.0 + _randn(g, (A, c["heads"], c["dk"]), 0.1),
        "beta": _randn(g, (A, c["heads"], c["dk"]), 0.05),
    }


# ---------------------------------------------------------------------------- the calls

def prepare(case, seed):
    c, i32, f32 = case, torch.int32, torch.float32
    if c["op"] == "query":
        s = _query_inputs(c, seed)
        qd = U.umem_query_desc()
        qd.d_model, qd.conv_k, qd.heads, qd.dk = c["d_model"], c["conv_k"], c["heads"], c["dk"]
        qd.shared, qd.eps = int(c["shared"]), 1e-5
        st, need = U.umem_query_workspace_size(qd, c["B"], c["L"])
        U.check(st)
        shape = (c["B"] * c["L"], c["heads"], c["dk"])
        s.update(case=c, desc=qd, ws=torch.empty(max(need, 256), dtype=torch.uint8, device=DEV),
                 q_row=torch.empty(shape, dtype=f32, device=DEV),
                 q_col=None if c["shared"] else torch.empty(shape, dtype=f32, device=DEV))
        return s
    s = _layer_inputs(c, seed)
    desc, T, H, m, h, dv = _desc(c), c["T"], c["heads"], c["topm"], _cores(c), c["dv"]
    s.update(case=c, desc=desc)
    wshape = (T, H, m) + ((h,) if h > 1 else ())
    if c["op"] == "forward":
        st, need = U.umem_workspace_size(desc, T)
        U.check(st)
        width = c["d_out"] or c["dv_virt"] or dv
        s.update(ws=torch.empty(max(need, 256), dtype=torch.uint8, device=DEV),
                 out=torch.empty((T, width), dtype=f32, device=DEV),
                 idx=torch.empty((T, H, m), dtype=i32, device=DEV),
                 # the scores of single-core layers are kept too, as a program that trains does
                 w=torch.empty(wshape, dtype=f32, device=DEV) if h == 1 else None)
        return s
    # the backward is given the forward's selection: here the exact one
    s.update(idx=None, w=None)
    s["idx"], w64 = _selection(c, s)
    s["w"] = w64.to(f32).contiguous()
    st, need_b = U.umem_gather_backward_workspace_size(T, _bag(c), dv)
    U.check(st)
    st, need_s = U.umem_score_backward_workspace_size(desc, T)
    U.check(st)
    M = T * _bag(c)
    s.update(ws=torch.empty(max(need_b, need_s, 256), dtype=torch.uint8, device=DEV),
             dw=torch.zeros(wshape, dtype=f32, device=DEV),
             dq_row=torch.zeros((T, H, c["dk"]), dtype=f32, device=DEV),
             dq_col=torch.zeros((T, H, c["dk"]), dtype=f32, device=DEV),
             dk_row=torch.zeros((H, c["n_keys"], c["dk"]), dtype=f32, device=DEV),
             dk_col=torch.zeros((H, c["n_keys"], c["dk"]), dtype=f32, device=DEV),
             dcore=torch.zeros_like(s["core"]) if c["rank"] else None)
    if c["dense"]:
        s.update(d_values=torch.zeros((_n_values(c), dv), dtype=f32, device=DEV))
    else:
        s.update(rows=torch.zeros((M,), dtype=i32, device=DEV),
                 d_rows=torch.zeros((M, dv), dtype=f32, device=DEV),
                 n_rows=torch.zeros((1,), dtype=i32, device=DEV))
    return s


def run(state):
    s, c, d = state, state["case"], state["desc"]
    ws = s["ws"]
    if c["op"] == "query":
        U.check(U.umem_query(d, c["B"], c["L"], s["x"], s["hist"], s["conv_w"], s["w_q"], s["gamma"],
                             s["beta"], s["q_row"], s["q_col"], ws, ws.numel()), "umem_query")
        return {"q_row": s["q_row"], "q_col": s["q_col"]}
    if c["op"] == "forward":
        U.check(U.umem_forward(d, c["T"], s["q_row"], s["q_col"], s["k_row"], s["k_col"], s["core"],
                               s["values"], s["perm"], s["w_proj"], s["w_out"], s["out"], s["idx"],
                               s["w"], ws, ws.numel()), "umem_forward")
        return {"out": s["out"], "idx": s["idx"], "w": s["w"]}
    # gradients that the library adds into are cleared, as between two steps of an optimiser
    s["dk_row"].zero_()
    s["dk_col"].zero_()
    if s["dcore"] is not None:
        s["dcore"].zero_()
    common = (d.n_values, d.dv, d.vdtype, s["values"], c["T"], _bag(c), s["idx"], s["w"], s["perm"],
              c["expand"], c["cores"], s["d_pooled"])
    if c["dense"]:
        s["d_values"].zero_()
        U.check(U.umem_gather_backward(*common, s["d_values"], s["dw"], ws, ws.numel()),
                "umem_gather_backward")
        got = {"d_values": s["d_values"]}
    else:
        U.check(U.umem_gather_backward_rows(*common, s["rows"], s["d_rows"], s["n_rows"], s["dw"], ws,
                                            ws.numel()), "umem_gather_backward_rows")
        got = {"rows": s["rows"], "d_rows": s["d_rows"], "n_rows": s["n_rows"]}
    U.check(U.umem_score_backward(d, c["T"], s["q_row"], s["q_col"], s["k_row"], s["k_col"], s["core"],
                                  s["idx"], s["w"], s["dw"], s["dq_row"], s["dq_col"], s["dk_row"],
                                  s["dk_col"], s["dcore"], ws, ws.numel()), "umem_score_backward")
    got.update({k: s[k] for k in ("dw", "dq_row", "dq_col", "dk_row", "dk_col", "dcore")})
    return got


# ---------------------------------------------------------------------------- what it takes

def _distinct_rows(c):
    """Value rows a call touches: uniform draws over the table, or tokens that share their
    cluster's slots (about four times a head's top-m for each cluster)."""
    N, M = _n_values(c), c["T"] * _bag(c)
    if c["clusters"]:
        M = min(M, 4 * c["clusters"] * _bag(c))
    return N * -math.expm1(-M / N)


def work(case):
    c = case
    if c["op"] == "query":
        T, nq = c["B"] * c["L"], (1 if c["shared"] else 2) * c["heads"] * c["dk"]
        rows = T + (c["B"] * (c["conv_k"] - 1) if c["history"] else 0)
        return {"bytes": 4 * rows * c["d_model"] + 2 * c["d_model"] * nq + 4 * T * nq,
                "flops": 2 * T * c["d_model"] * (nq + c["conv_k"])}
    T, H, n, dk, dv, E, h = c["T"], c["heads"], c["n_keys"], c["dk"], c["dv"], c["expand"], _cores(c)
    esize = 2 if c["bf16"] else 4
    bag, rows = _bag(c), _distinct_rows(c)
    qk = 4 * 2 * H * dk * (T + n)
    sel = T * bag * 4 * (1 + h)
    if c["op"] == "forward":
        k1 = E * dv
        weights = 2 * (c["dv_virt"] * k1 + c["d_out"] * (c["dv_virt"] or dv))
        out = 4 * T * (c["d_out"] or c["dv_virt"] or dv)
        return {"bytes": qk + rows * dv * esize + sel + weights + out,
                "flops": 4 * T * H * n * dk + 2 * T * bag * dv + T * weights}
    # selected keys are read, key gradients of the selected keys written; rows read, gradients
    # written (a dense table is cleared as well)
    keys = min(n, T * c["topm"])
    grads = 2 * rows * dv * 4 + _n_values(c) * dv * 4 if c["dense"] else rows * (dv * 4 + 4)
    return {"bytes": rows * dv * esize + grads + T * E * dv * 4 + sel + 4 * T * bag * h
            + 4 * 2 * H * dk * (2 * T + 2 * keys),
            "flops": 4 * T * bag * dv + 8 * T * bag * dk}


def tolerance(case):
    c = case
    if c["op"] == "query":
        # convolved rows rounded to bf16 before the linear; a sum in another order moves some of
        # those roundings by one step
        return {"rel": 1e-3, "max": 2e-2}
    if c["op"] == "backward":
        return {"rel": 1e-5, "max": 1e-3}                 # sums of fp32 products
    # Selected scores that agree to fp32's last bits may come in the other order (differ), and the
    # last selected slot of a few tokens in a thousand may be the next one.
    few = c["T"] * c["heads"] >= 256
    if c["d_out"] or c["dv_virt"]:
        return {"rel": 1e-2, "max": 0.99 if few else 0.1, "differ": 1e-3}   # bf16 GEMM operands
    return {"rel": 1e-2 if few else 1e-5, "max": 0.99 if few else 1e-3, "differ": 1e-3}


# ---------------------------------------------------------------------------- float64 reference

def _factors(core, cores):
    """Leading singular pair (u, t) of each head's core, u's largest component positive."""
    C = core.double()
    C = C.sum(dim=1) if cores > 1 else C
    A, _, B = torch.linalg.svd(C.cpu())
    u, t = A[:, :, 0], B[:, 0, :]
    sign = torch.sign(torch.gather(u, 1, u.abs().argmax(dim=1, keepdim=True)))
    return (u * sign).to(DEV), (t * sign).to(DEV), C


def _selection(c, s):
    """(idx int32 [T, H, m], weights float64 [T, H, m] or [T, H, m, cores]), best score first."""
    T, H, n, k, m, r = c["T"], c["heads"], c["n_keys"], c["topk"], c["topm"], c["rank"]
    idx = torch.empty((T, H, m), dtype=torch.int32, device=DEV)
    h = _cores(c)
    w = torch.empty((T, H, m) + ((h,) if h > 1 else ()), dtype=torch.float64, device=DEV)
    if r:
        u, t, C = _factors(s["core"], c["cores"])
    for head in range(H):
        S = []                                   # per axis [T, r or 1, n]
        for q, K in ((s["q_row"], s["k_row"]), (s["q_col"], s["k_col"])):
            qh, Kh = q[:, head].double(), K[head].double()
            width = c["dk"] // max(1, r)
            S.append([qh[:, x * width:(x + 1) * width] @ Kh[:, x * width:(x + 1) * width].t().contiguous()
                      for x in range(max(1, r))])
        fold = [[1.0], [1.0]] if not r else [u[head], t[head]]
        top, at = [], []
        for a in range(2):
            score = sum(f * x for f, x in zip(fold[a], S[a]))
            i = torch.topk(score, k, dim=1).indices
            top.append(i)
            at.append([x.gather(1, i) for x in S[a]])          # [T, k] per slice
        if not r:
            grid = at[0][0][:, :, None] + at[1][0][:, None, :]
        else:
            p = [sum(C[head, x, y] * at[1][y] for y in range(r)) for x in range(r)]
            grid = sum(at[0][x][:, :, None] * p[x][:, None, :] for x in range(r))
        best = torch.topk(grid.reshape(T, k * k), m, dim=1)
        a, b = best.indices // k, best.indices % k
        idx[:, head] = (top[0].gather(1, a) * n + top[1].gather(1, b)).to(torch.int32)
        if h > 1:
            for x in range(h):
                Cx = s["core"][head, x].double()
                w[:, head, :, x] = sum(at[0][i].gather(1, a) * sum(Cx[i, j] * at[1][j].gather(1, b) for j in range(r))
                                       for i in range(r))
        elif c["softmax"]:
            w[:, head] = torch.softmax(best.values, dim=1)
        else:
            w[:, head] = best.values
    return idx, w


def _slots(c, s, idx):
    """Virtual block and physical row of each bag entry, [T, bag] each."""
    flat = idx.reshape(c["T"], _bag(c)).long()
    if c["expand"] > 1:
        flat = s["perm"].long()[flat]
    N = _n_values(c)
    return flat // N, flat % N


def _per_core(c, w):
    return w.reshape(c["T"], _bag(c), _cores(c))


def _exact_forward(c, s):
    idx, w = _selection(c, s)
    T, E, dv, h = c["T"], c["expand"], c["dv"], _cores(c)
    block, row = _slots(c, s, idx)
    wc = _per_core(c, w)
    pooled = torch.zeros((T, E, dv), dtype=torch.float64, device=DEV)
    step = max(1, (1 << 27) // (_bag(c) * dv))
    for t0 in range(0, T, step):
        ts = slice(t0, t0 + step)
        V = s["values"][row[ts]].double()                       # [t, bag, dv]
        for x in range(h):
            cols = slice(x * dv // h, (x + 1) * dv // h)
            Vx = V[:, :, cols].contiguous()
            for p in range(E):
                wp = torch.where(block[ts] == p, wc[ts, :, x], 0.0)
                pooled[ts, p, cols] = torch.matmul(wp[:, None, :], Vx)[:, 0]
    out = pooled.reshape(T, E * dv)
    for weight in (s["w_proj"], s["w_out"]):
        if weight is not None:
            out = out @ weight.double().t().contiguous()
    return {"out": out, "idx": None, "w": w if h == 1 else None}


def _exact_backward(c, s):
    T, H, m, E, dv, dk, h, r = (c["T"], c["heads"], c["topm"], c["expand"], c["dv"], c["dk"], _cores(c),
                                c["rank"])
    bag, n = _bag(c), c["n_keys"]
    idx, w64 = _selection(c, s)
    w = _per_core(c, w64.to(torch.float32).double())
    block, row = _slots(c, s, idx)
    uniq, inv = torch.unique(row.reshape(-1), return_inverse=True)
    inv = inv.reshape(T, bag)
    d_rows = torch.zeros((len(uniq), dv), dtype=torch.float64, device=DEV)
    dw = torch.empty((T, bag, h), dtype=torch.float64, device=DEV)
    step = max(1, (1 << 26) // (bag * dv))
    for t0 in range(0, T, step):
        ts = slice(t0, min(T, t0 + step))
        tt = torch.arange(ts.start, ts.stop, device=DEV)[:, None]
        dp = s["d_pooled"][tt, block[ts]].double()               # [t, bag, dv]
        V = s["values"][row[ts]].double()
        dw[ts] = (dp * V).reshape(-1, bag, h, dv // h).sum(dim=3)
        add = dp.reshape(-1, bag, h, dv // h) * w[ts, :, :, None]
        d_rows.index_add_(0, inv[ts].reshape(-1), add.reshape(-1, dv))
    got = {}
    if c["dense"]:
        got["d_values"] = torch.zeros((_n_values(c), dv), dtype=torch.float64, device=DEV)
        got["d_values"][uniq] = d_rows
    else:
        got.update(rows=None, n_rows=None)
        got["d_rows"] = torch.zeros((T * bag, dv), dtype=torch.float64, device=DEV)
        got["d_rows"][:len(uniq)] = d_rows
    dg = dw.reshape(T, H, m, h)
    got["dw"] = dg if h > 1 else dg[..., 0]
    if c["softmax"]:
        ww = w.reshape(T, H, m, h)
        dg = ww * (dg - (ww * dg).sum(dim=2, keepdim=True))
    ij = (idx.long() // n, idx.long() % n)
    heads = torch.arange(H, device=DEV)[None, :, None]
    R = max(1, r)
    K = [k[heads, x].double().reshape(T, H, m, R, dk // R)
         for k, x in zip((s["k_row"], s["k_col"]), ij)]
    q = [x.double().reshape(T, H, R, dk // R) for x in (s["q_row"], s["q_col"])]
    if r:
        S = [(k * x[:, :, None]).sum(dim=4) for k, x in zip(K, q)]             # [T, H, m, r]
        C = s["core"].double().reshape(1, H, 1, h, r, r)
        CS = [(C * S[1][:, :, :, None, None, :]).sum(dim=5),                   # [T, H, m, h, r]
              (C * S[0][:, :, :, None, :, None]).sum(dim=4)]
        dS = [(dg[..., None] * x).sum(dim=3) for x in CS]                      # [T, H, m, r]
        outer = S[0][:, :, :, :, None] * S[1][:, :, :, None, :]                # [T, H, m, r, r]
        dC = torch.stack([(dg[..., x, None, None] * outer).sum(dim=(0, 2)) for x in range(h)], dim=1)
        got["dcore"] = dC if h > 1 else dC[:, 0]
    else:
        dS = [dg, dg]
        got["dcore"] = None
    for name, a in (("row", 0), ("col", 1)):
        got["dq_" + name] = (dS[a][..., None] * K[a]).sum(dim=2).reshape(T, H, dk)
        add = dS[a][..., None] * q[a][:, :, None]                              # [T, H, m, R, w]
        dK = torch.zeros((H * n, dk), dtype=torch.float64, device=DEV)
        dK.index_add_(0, (heads * n + ij[a]).reshape(-1), add.reshape(-1, dk))
        got["dk_" + name] = dK.reshape(H, n, dk)
    return got


def _exact_query(c, s):
    B, L, d, kc = c["B"], c["L"], c["d_model"], c["conv_k"]
    x = s["x"].double()
    past = s["hist"].double() if s["hist"] is not None else torch.zeros((B, kc - 1, d), dtype=torch.float64, device=DEV)
    full = torch.cat([past, x], dim=1)
    y = sum(s["conv_w"][j].double() * full[:, kc - 1 - j:kc - 1 - j + L] for j in range(kc))
    q = y.reshape(B * L, d) @ s["w_q"].double().t().contiguous()
    A = 1 if c["shared"] else 2
    q = q.reshape(B * L, A, c["heads"], c["dk"])
    q = (q - q.mean(dim=3, keepdim=True)) / torch.sqrt(q.var(dim=3, unbiased=False, keepdim=True) + 1e-5)
    q = q * s["gamma"].double() + s["beta"].double()
    return {"q_row": q[:, 0].contiguous(), "q_col": None if c["shared"] else q[:, 1].contiguous()}


def exact(case, seed):
    if case["op"] == "query":
        return _exact_query(case, _query_inputs(case, seed))
    s = _layer_inputs(case, seed)
    return _exact_forward(case, s) if case["op"] == "forward" else _exact_backward(case, s)
