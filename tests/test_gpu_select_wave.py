"""The selection that gives each (token, head) pair one wave (2,048 pairs and more, 8,192 beyond 2,048
keys) against the one that gives it a workgroup: the same slots, weights and per-axis indices,
bit for bit, on every form both take.  The workgroup kernel, itself held to the oracle, is reached by
selecting the same scores a few hundred tokens at a time."""
from __future__ import annotations

import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():     # collected on CPU hosts too; every test here is gpu-marked
    pytest.skip("no GPU", allow_module_level=True)

import paper_2411_12364_amd as U                    # noqa: E402
from synth import configs as CF                     # noqa: E402
from tests import gpu_util as G                     # noqa: E402


def layer(T, heads, n, k, m, rank=0, cores=1, dk=64, softmax=False):
    return CF.Layer("select-wave", T=T, heads=heads, dk=dk, n_keys=n, topk=k, topm=m, dv=64,
                    vdtype=CF.BF16, seed=0, rank=max(1, rank),
                    grid=CF.GRID_TUCKER if rank else CF.GRID_ADD,
                    weight=CF.W_SOFTMAX if softmax else CF.W_RAW, cores=cores)


def select(cfg, T, sel, q, K, core, axis):
    desc = G.desc_for(cfg)
    idx = torch.empty((T, cfg.heads, cfg.topm), dtype=torch.int32, device="cuda")
    w = torch.empty(G.weights_shape(cfg, T), dtype=torch.float32, device="cuda")
    ax = torch.empty((2, T, cfg.heads, cfg.topk), dtype=torch.int32, device="cuda") if axis else None
    tucker = cfg.grid == CF.GRID_TUCKER
    U.check(U.umem_select(desc, T, sel, *(q if tucker else (None, None)), *(K if tucker else (None, None)),
                          core, idx, w, ax), "umem_select")
    return idx, w, ax


def check(cfg, sel, q, K, core, axis):
    T, step = cfg.T, 2047 // cfg.heads              # a step stays below 2,048 pairs
    idx, w, ax = select(cfg, T, sel, q, K, core, axis)
    for t0 in range(0, T, step):
        ts = slice(t0, min(T, t0 + step))
        n = ts.stop - t0
        i2, w2, a2 = select(cfg, n, sel[:, ts].contiguous(), [x[ts].contiguous() for x in q], K, core, axis)
        assert torch.equal(idx[ts], i2)
        nan = w2.isnan()                            # (a NaN's payload says nothing)
        assert torch.equal(w[ts].isnan(), nan)
        assert torch.equal(w[ts][~nan].view(torch.int32), w2[~nan].view(torch.int32))
        if axis:
            assert torch.equal(ax[:, ts], a2)


def scores(kind, cfg, g):
    sel = torch.randn((2, cfg.T, cfg.heads, cfg.n_keys), device="cuda", generator=g)
    if kind == "ties":                                # some 30 distinct values: massive ties
        sel = (sel * 4).round() / 4
    elif kind == "few ties":                          # groups of a few equal scores
        sel = sel.bfloat16().float()
    elif kind == "twins":                             # every score twice, every pair four times
        sel[..., 1::2] = sel[..., ::2]
    elif kind == "equal":
        sel.zero_()
        sel[:, 1::2] = -0.0
    elif kind == "few":                               # fewer numbers than the top-k, the rest NaN
        sel[..., cfg.topk // 2:] = float("nan")
    elif kind == "inf":
        sel[..., ::3] = float("-inf")
        sel[:, ::5, :, 7] = float("inf")
        sel[:, ::7, :, 11] = float("nan")
    elif kind == "masked":                            # -inf but for a few keys: fewer than the top-k, then
        sel[:, ::2, :, max(1, cfg.topk // 2):] = float("-inf")             # more, on few lanes
        sel[:, 1::2, :, 100:] = float("-inf")
    elif kind == "all masked":
        sel[..., :] = float("-inf")
        sel[:, ::3, :, 5:9] = float("nan")
    elif kind == "opposite":                          # rows of +inf, columns of -inf: the grid's pairs
        sel[0, ..., : min(cfg.topk, cfg.topm) - 1] = float("inf")     # are NaN in all the candidates' rows but one
        sel[1] = float("-inf")
    elif kind == "lowest":                            # a mask of the type's lowest value
        sel[..., 3:] = torch.finfo(torch.float32).min
    return sel


# n: one 256-key step to eighteen, remainders of 4 and of 252; k, m: 1, the largest, m > k
ADDITIVE = [(2048, 1, 512, 32, 32), (1030, 2, 1024, 33, 64), (700, 3, 772, 1, 1), (4100, 2, 2308, 20, 17),
            (4097, 2, 4480, 32, 32), (2049, 1, 2044, 60, 40)]
OPPOSITE = [(2048, 1, 512, 2, 2), (2048, 1, 512, 32, 32), (1030, 2, 1024, 33, 64), (2049, 1, 2044, 60, 40)]


@pytest.mark.parametrize("kind", ["normal", "ties", "few ties", "twins", "equal", "few", "inf", "lowest", "masked", "all masked"])
@pytest.mark.parametrize("T,heads,n,k,m", ADDITIVE)
def test_additive(T, heads, n, k, m, kind):
    print(f"[case] wave additive T={T} H={heads} n={n} k={k} m={m} {kind}", flush=True)
    cfg = layer(T, heads, n, k, m, softmax=(kind == "normal" and k % 2 == 0))
    g = torch.Generator(device="cuda").manual_seed(n + k)
    check(cfg, scores(kind, cfg, g), [torch.empty(0)] * 2, None, None, axis=(m != 17))


@pytest.mark.parametrize("T,heads,n,k,m", OPPOSITE)
def test_additive_opposite_infinities(T, heads, n, k, m):
    """Every slot is written, with a candidate of its own, where most of the grid is +inf - inf: the best
    is the finite row's first column, the others NaN or -inf."""
    print(f"[case] wave additive opposite infinities T={T} H={heads} n={n} k={k} m={m}", flush=True)
    cfg = layer(T, heads, n, k, m)
    g = torch.Generator(device="cuda").manual_seed(n + k)
    sel = scores("opposite", cfg, g)
    check(cfg, sel, [torch.empty(0)] * 2, None, None, axis=True)
    for ts in (slice(0, T), slice(0, 5)):             # either kernel
        idx, w, ax = select(cfg, ts.stop, sel[:, ts].contiguous(), [torch.empty(0)] * 2, None, None, True)
        assert torch.equal(idx[..., 0], ax[0, ..., min(k, m) - 1] * n + ax[1, ..., 0])
        assert bool((w[..., 0] == float("-inf")).all()) and bool((w.isnan() | w.isneginf()).all())
        assert bool(((idx >= 0) & (idx < n * n)).all())
        assert all(x.unique().numel() == m for x in idx[:3].reshape(-1, m))


# (T, heads, n, k, m, rank, cores, dk): whole and ragged batches of key pieces, k and m from one to
# the largest, and a core close to rank one (most of the best in a few columns)
TUCKER = [(512, 4, 2048, 64, 64, 2, 1, 128), (1024, 2, 1792, 42, 42, 2, 2, 448), (2051, 1, 512, 7, 33, 2, 1, 24),
          (700, 3, 1020, 16, 1, 1, 1, 20), (1024, 2, 2048, 64, 64, 1, 1, 64), (4097, 2, 4480, 30, 50, 2, 4, 40)]


@pytest.mark.parametrize("kind", ["normal", "ties", "twins", "zero", "near-rank-1", "nan", "masked", "all masked", "huge",
                                  "overflow"])
@pytest.mark.parametrize("T,heads,n,k,m,rank,cores,dk", TUCKER)
def test_tucker(T, heads, n, k, m, rank, cores, dk, kind):
    print(f"[case] wave Tucker T={T} H={heads} n={n} k={k} m={m} r={rank} h={cores} dk={dk} {kind}", flush=True)
    cfg = layer(T, heads, n, k, m, rank, cores, dk, softmax=(kind == "normal" and cores == 1))
    g = torch.Generator(device="cuda").manual_seed(n + k + dk)
    rnd = lambda *shape: torch.randn(shape, device="cuda", generator=g)     # noqa: E731
    q = [rnd(T, heads, dk), rnd(T, heads, dk)]
    K = [rnd(heads, n, dk), rnd(heads, n, dk)]
    core = rnd(heads, cores, rank, rank) if cores > 1 else rnd(heads, rank, rank)
    if kind == "ties":
        q = [x.sign() for x in q]
        K = [x.sign() for x in K]
        core = core.sign()
    elif kind == "twins":                             # every key twice
        for x in K:
            x[:, 1::2] = x[:, ::2]
    elif kind == "zero":                              # padding tokens
        q[0][::2] = 0.0
        q[1][::3] = 0.0
    elif kind == "near-rank-1":
        core.fill_(1.0)
        core[..., 0, 0] += 1e-3
    elif kind == "nan":
        q[0][::3] = float("nan")
        K[1][:, ::2] = float("nan")
    elif kind == "huge":                              # grid scores beyond fp32: all below, or all but one
        q = [x.abs() * 1e18 for x in q]               # column's
        K = [x.abs() * 1e18 for x in K]
        K[1][1:, 5] *= -1.5
        core.fill_(-1.0)
    elif kind == "overflow":                          # per-slice scores beyond fp32
        q = [x * 1e20 for x in q]
        K = [x * 1e20 for x in K]
    width = dk // rank
    sel = torch.stack([sum(torch.einsum("thd,hnd->thn", x[..., r * width:(r + 1) * width].double(),
                                        y[..., r * width:(r + 1) * width].double()) for r in range(rank)).float()
                       for x, y in zip(q, K)])
    if kind == "huge":
        sel.abs_()
    if kind.endswith("masked"):                       # as "masked" and "all masked" above
        sel = torch.minimum(sel, scores(kind, cfg, g))
    check(cfg, sel.contiguous(), q, K, core, axis=(k % 2 == 1))
