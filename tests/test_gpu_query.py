"""GPU parity of the query front-end and the key LayerNorm through the C ABI, against the
front-end oracle on the same seeded inputs; and the layer fed end to end with the queries and
keys they produce."""
from __future__ import annotations

import dataclasses
import sys

import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():     # collected on CPU hosts too; every test here is gpu-marked
    pytest.skip("no GPU", allow_module_level=True)

import oracle.query_oracle as Q                     # noqa: E402
import paper_2411_12364_amd as U                    # noqa: E402
import synth as S                                   # noqa: E402
from synth import configs as CF                     # noqa: E402
from synth import device as SD                      # noqa: E402
from tests import gpu_util as G                     # noqa: E402
from tests import parity as P                       # noqa: E402

# Query rows: bf16 rounding of the convolved rows before the linear (relative 2^-9 per element)
# gives about 1e-3 of a row's scale after the LayerNorm; the bound leaves a 10x margin.
Q_RTOL = 1e-2


def log(*a):
    print(*a, flush=True)
    sys.stdout.flush()


def qdesc(fe):
    d = U.umem_query_desc()
    d.d_model, d.conv_k, d.heads, d.dk = fe.d_model, fe.conv_k, fe.heads, fe.dk
    d.shared, d.eps = int(fe.shared), fe.eps
    return d


def run_query(fe, inp=None):
    inp = inp or CF.front_end_inputs(fe)
    qd = qdesc(fe)
    st, nws = U.umem_query_workspace_size(qd, fe.B, fe.L)
    U.check(st)
    ws = torch.empty(max(nws, 256), dtype=torch.uint8, device="cuda")
    dev = lambda a: None if a is None else torch.from_numpy(np.ascontiguousarray(a)).cuda()
    q_row = torch.empty((fe.T, fe.heads, fe.dk), dtype=torch.float32, device="cuda")
    q_col = None if fe.shared else torch.empty_like(q_row)
    log(f"[case] query front-end {fe.name}: B={fe.B} L={fe.L} d={fe.d_model} K_c={fe.conv_k} "
        f"H={fe.heads} Dk={fe.dk} shared={fe.shared}")
    U.check(U.umem_query(qd, fe.B, fe.L, dev(inp["x"]), dev(inp["hist"]), dev(inp["conv_w"]),
                         dev(CF.output_major(inp["w_q"]).view(np.int16)), dev(inp["gamma"]), dev(inp["beta"]),
                         q_row, q_col, ws, ws.numel()), "umem_query")
    torch.cuda.synchronize()
    return inp, q_row, (q_row if fe.shared else q_col), ws


def oracle_queries(fe, inp):
    wq = S.bf16_bits_to_f32(inp["w_q"]).reshape(inp["w_q"].shape)
    return Q.query_front_end(inp["x"], inp["conv_w"], wq, inp["gamma"], inp["beta"], fe.heads,
                             fe.dk, fe.shared, inp["hist"], fe.eps)


def rounded_rows_queries(fe, inp):
    """The oracle's steps with the query linear's documented input rounding (the convolved rows
    to bf16, nearest even) applied to the oracle's own fp64 convolution: [T, A, H, Dk]."""
    A = 1 if fe.shared else 2
    wq = S.bf16_bits_to_f32(inp["w_q"]).reshape(inp["w_q"].shape).astype(np.float64)
    y = Q.causal_conv(inp["x"], inp["conv_w"], inp["hist"]).reshape(fe.T, fe.d_model)
    y16 = S.bf16_bits_to_f32(S.f32_to_bf16_bits(y.astype(np.float32))).reshape(y.shape)
    lin = Q.query_linear(y16.astype(np.float64), wq).reshape(fe.T, A, fe.heads, fe.dk)
    g = np.asarray(inp["gamma"], np.float64).reshape(A, fe.heads, fe.dk)
    b = np.asarray(inp["beta"], np.float64).reshape(A, fe.heads, fe.dk)
    return Q.layer_norm(lin, g, b, fe.eps)


ROUNDED_RTOL = 2e-3   # fp32 accumulation, and a rare bf16 rounding decided the other way


def row_err(got, ref):
    got = np.asarray(got, np.float64).reshape(-1, ref.shape[-1])
    ref = np.asarray(ref, np.float64).reshape(-1, ref.shape[-1])
    return float((np.abs(got - ref).max(axis=1) / np.abs(ref).max(axis=1)).max())


CASES = [
    CF.FrontEnd("small-shared", B=2, L=5, d_model=64, conv_k=4, heads=2, dk=64, shared=True, seed=21),
    CF.FrontEnd("separate-start", B=3, L=7, d_model=96, conv_k=3, heads=1, dk=40, shared=False,
                seed=22, history=False),
    CF.FrontEnd("single-tap", B=4, L=2, d_model=128, conv_k=1, heads=2, dk=128, shared=True, seed=23),
    CF.FE6,
    CF.FrontEnd("prefill-chunk", B=2, L=300, d_model=1024, conv_k=4, heads=2, dk=128, shared=False,
                seed=24),
    # the limits: eight taps, Dk = 1024 (16 values per lane in the LayerNorm, which then adds
    # the query linear's 8 split partials in two batches)
    CF.FrontEnd("limits", B=3, L=9, d_model=2048, conv_k=8, heads=2, dk=1024, shared=False, seed=25),
]


@pytest.mark.parametrize("kc", range(1, 9))
def test_convolution_runs(kc):
    """Runs of four tokens to a thread (2,048 tokens and more): every tap count, runs that cross from
    one sequence into the next and end past the last token, with and without a history.  Half a bf16
    step (2^-8 of the value) and the fp32 sum's error (kc products of order one)."""
    fe = CF.FrontEnd(f"conv-runs-{kc}", B=3, L=709, d_model=72, conv_k=kc, heads=1, dk=8, shared=True,
                     seed=30 + kc, history=kc % 2 == 0)
    inp, _, _, ws = run_query(fe)
    y = torch.empty(fe.T * fe.d_model, dtype=torch.int16)
    y.copy_(ws[: fe.T * fe.d_model * 2].view(torch.int16))
    got = S.bf16_bits_to_f32(y.numpy().view(np.uint16)).reshape(fe.T, fe.d_model).astype(np.float64)
    ref = Q.causal_conv(inp["x"], inp["conv_w"], inp["hist"]).reshape(fe.T, fe.d_model)
    assert (np.abs(got - ref) <= np.abs(ref) * 2.0 ** -8 + kc * 4 * 2.0 ** -23).all()


def test_convolution_past_one_launch():
    """2^20 sequences of one token over 16,384 channels: more threads than one launch of the convolution
    takes.  Tokens at the ends and at the bands' edges (2^19 runs each) against fp64 (half a bf16 step
    and the fp32 sum's error)."""
    T, d = 1 << 20, 16384
    if torch.cuda.mem_get_info()[0] < 120 << 30:
        pytest.skip("needs 120 GiB of device memory")
    log(f"[case] convolution past one launch: T={T} d={d}")
    qd = U.umem_query_desc()
    qd.d_model, qd.conv_k, qd.heads, qd.dk, qd.shared, qd.eps = d, 1, 1, 8, 1, 1e-5
    st, nws = U.umem_query_workspace_size(qd, T, 1)
    U.check(st)
    g = torch.Generator(device="cuda").manual_seed(5)
    ws = torch.empty(nws, dtype=torch.uint8, device="cuda")
    ws[: T * d * 2].view(torch.int16).fill_(0x7FC0)       # NaN where no token is written
    x = torch.empty((T, 1, d), dtype=torch.float32, device="cuda").normal_(generator=g)
    w = torch.randn((1, d), device="cuda", generator=g)
    wq = torch.randn((8, d), device="cuda", generator=g).to(torch.bfloat16)
    q = torch.empty((T, 1, 8), dtype=torch.float32, device="cuda")
    U.check(U.umem_query(qd, T, 1, x, None, w, wq.view(torch.int16), torch.ones((1, 1, 8), device="cuda"),
                         torch.zeros((1, 1, 8), device="cuda"), q, None, ws, ws.numel()), "umem_query")
    torch.cuda.synchronize()
    y = ws[: T * d * 2].view(torch.bfloat16).view(T, d)
    for t in (0, 1, T // 2 - 1, T // 2, T // 2 + 1, T - 1):
        ref = x[t, 0].double() * w[0].double()
        assert bool(((y[t].double() - ref).abs() <= ref.abs() * 2.0 ** -8 + 4 * 2.0 ** -23).all()), t
    assert not bool(y[:, ::4096].isnan().any())
    assert not bool(q.isnan().any())
    del x, ws, y
    torch.cuda.empty_cache()


@pytest.mark.parametrize("T,K,N", [(1, 8, 8), (63, 520, 72), (65, 2048, 64), (130, 1024, 200),
                                   (2036, 2048, 512), (65, 2056, 72), (2036, 1536, 2040),
                                   (2036, 1544, 2040)])
def test_small_tiles(T, K, N):
    """The 64 x 64 tiles of short products (K <= 2048, too few 128 x 128 tiles for the chip; K <= 1536 from
    256 such tiles on) at their edges, and just past the rule: against fp64 on the bf16-rounded operands, within the bound of an
    fp32 sum of K products (K 2^-23 of the sum of their magnitudes)."""
    log(f"[case] small tiles T={T} K={K} N={N}")
    g = torch.Generator(device="cuda").manual_seed(T + K + N)
    a = torch.randn((T, 1, K), device="cuda", generator=g)
    b = torch.randn((N, K), device="cuda", generator=g).to(torch.bfloat16)
    out = torch.empty((T, N), device="cuda")
    st, nws = U.umem_project_workspace_size(T, 1, K, 0, N)
    U.check(st)
    ws = torch.empty(max(nws, 256), dtype=torch.uint8, device="cuda")
    U.check(U.umem_project(T, 1, K, 0, N, a, None, b.view(torch.int16), out, ws, ws.numel()))
    torch.cuda.synchronize()
    A = a[:, 0].to(torch.bfloat16).double()
    Bt = b.double().t().contiguous()
    bound = K * 2.0 ** -23 * (A.abs() @ Bt.abs())
    assert bool(((out.double() - A @ Bt).abs() <= bound).all())


@pytest.mark.parametrize("fe", CASES, ids=[c.name for c in CASES])
def test_query_front_end(fe):
    inp, q_row, q_col, ws = run_query(fe)
    # the convolution: the first T * d bf16 values of the workspace (fp32 sums rounded to bf16,
    # against fp64): within half a bf16 step of the exact value (bf16 carries 8 significant bits:
    # at most 2^-8 relative), plus the fp32 sum's own error
    y16 = ws[: fe.T * fe.d_model * 2].view(torch.int16).cpu().numpy()
    y = S.bf16_bits_to_f32(y16).reshape(fe.B, fe.L, fe.d_model).astype(np.float64)
    y_ref = Q.causal_conv(inp["x"], inp["conv_w"], inp["hist"])
    bound = 2.0 ** -8 * np.abs(y_ref) + 1e-6 * np.abs(y_ref).max()
    conv_err = float(np.abs(y - y_ref).max() / np.abs(y_ref).max())
    assert np.all(np.abs(y - y_ref) <= bound), conv_err
    qr_ref, qc_ref = oracle_queries(fe, inp)
    er, ec = row_err(q_row.cpu().numpy(), qr_ref), row_err(q_col.cpu().numpy(), qc_ref)
    r16 = rounded_rows_queries(fe, inp)
    e16 = max(row_err(q.cpu().numpy(), r16[:, 0 if fe.shared else a]) for a, q in enumerate((q_row, q_col)))
    log(f"[report] {fe.name}: conv err {conv_err:.2e}, q_row err {er:.2e}, q_col err {ec:.2e}, "
        f"against bf16-rounded rows {e16:.2e}")
    assert er <= Q_RTOL and ec <= Q_RTOL and e16 <= ROUNDED_RTOL


def test_query_deterministic():
    fe = CF.FE6
    inp, a, _, _ = run_query(fe)
    _, b, _, _ = run_query(fe, inp)
    assert torch.equal(a, b)


def test_query_graph_replay_stale_workspace():
    """The 1.6B-x12 front-end (convolution, split-K query linear, LayerNorm) captured in a HIP
    graph and replayed over a garbage-filled workspace, with eager work between replays, gives
    the eager queries bit for bit."""
    fe = CF.FE6
    inp = CF.front_end_inputs(fe)
    qd = qdesc(fe)
    st, nws = U.umem_query_workspace_size(qd, fe.B, fe.L)
    U.check(st)
    ws = torch.empty(max(nws, 256), dtype=torch.uint8, device="cuda")
    dev = lambda a: None if a is None else torch.from_numpy(np.ascontiguousarray(a)).cuda()
    x, hist, cw = dev(inp["x"]), dev(inp["hist"]), dev(inp["conv_w"])
    wq = dev(CF.output_major(inp["w_q"]).view(np.int16))
    g_, b_ = dev(inp["gamma"]), dev(inp["beta"])
    q_row = torch.empty((fe.T, fe.heads, fe.dk), dtype=torch.float32, device="cuda")
    q_col = None if fe.shared else torch.empty_like(q_row)

    def step():
        U.check(U.umem_query(qd, fe.B, fe.L, x, hist, cw, wq, g_, b_, q_row, q_col, ws, ws.numel()),
                "umem_query")

    step()
    torch.cuda.synchronize()
    want = q_row.clone()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        step()
    for rep in range(4):
        q_row.fill_(-1.0)
        ws.fill_(0x3C)
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(q_row, want), rep
        step()
        torch.cuda.synchronize()


@pytest.mark.parametrize("H,n,dk", [(2, 300, 64), (4, 2048, 128), (2, 1792, 448), (1, 5, 1000)])
def test_key_norm(H, n, dk):
    cfg = CF.Layer("keys", T=1, heads=H, dk=dk, n_keys=n, topk=1, topm=1, dv=8, vdtype=CF.F32, seed=40 + dk)
    kr, _ = CF.keys(cfg)
    g, b = CF.key_norm_params(cfg)
    keys = torch.from_numpy(kr).cuda()
    out = torch.empty_like(keys)
    U.check(U.umem_key_norm(H, n, dk, keys, torch.from_numpy(g).cuda(), torch.from_numpy(b).cuda(),
                            1e-5, out))
    torch.cuda.synchronize()
    ref = Q.key_norm(kr, g, b, 1e-5)
    err = row_err(out.cpu().numpy(), ref)
    log(f"[report] key norm H={H} n={n} dk={dk}: err {err:.2e}")
    assert err <= 1e-5
    # in place
    U.check(U.umem_key_norm(H, n, dk, keys, torch.from_numpy(g).cuda(), torch.from_numpy(b).cuda(),
                            1e-5, keys))
    torch.cuda.synchronize()
    assert torch.equal(keys, out)


def test_front_end_feeds_the_layer():
    """Queries from the front-end and LayerNormed keys drive the rank-2 Tucker layer with two
    component cores; the selection and pooling are checked against the oracle on those same
    queries and keys."""
    fe = CF.FrontEnd("e2e", B=4, L=8, d_model=128, conv_k=4, heads=2, dk=64, shared=True, seed=31)
    cfg = CF.Layer("e2e-layer", T=fe.T, heads=2, dk=64, n_keys=96, topk=16, topm=24, dv=512,
                   vdtype=CF.BF16, seed=31, rank=2, grid=CF.GRID_TUCKER, cores=2)
    _, q_row, q_col, _ = run_query(fe)
    dl = SD.make_layer(cfg)
    g, b = CF.key_norm_params(cfg)
    kr = torch.empty_like(dl.k_row)
    kc = torch.empty_like(dl.k_col)
    for src, dst in ((dl.k_row, kr), (dl.k_col, kc)):
        U.check(U.umem_key_norm(cfg.heads, cfg.n_keys, cfg.dk, src, torch.from_numpy(g).cuda(),
                                torch.from_numpy(b).cuda(), 1e-5, dst))
    dl = dataclasses.replace(dl, q_row=q_row[None], q_col=q_col[None], k_row=kr, k_col=kc)
    idx, w, ax = G.score_topk(dl, cfg.T, 0)
    pooled = G.gather(dl, idx, w, cfg.T)
    torch.cuda.synchronize()
    qh, kh = q_row.cpu().numpy(), (kr.cpu().numpy(), kc.cpu().numpy())
    _, rep = P.check_selection(cfg, qh, qh, kh[0], kh[1], CF.core(cfg), G.host(idx), G.host(w),
                               G.host(ax))
    _, err = P.check_pooled(cfg, G.value_rows_fn(cfg), G.host(idx), G.host(w), G.host(pooled))
    log(f"[report] front-end -> layer: {rep}, pooled err {err:.2e}")
