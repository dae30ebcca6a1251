"""GPU parity of the one-pass attention's gradients (zeta_select_attend_bwd)
against the float64 oracle (Appendix E.2), for the windows the one-pass call
selects (the same windows, bit for bit, as the oracle's selection).

Tolerance as for zeta_topk_attn_bwd: max-abs error at most
1e-4 * (1 + max |oracle|) per tensor, relative 1e-4 for the eps gradient.
The attention weights reach dv through two bfloat16 parts (16 significant
bits), far inside that bound.
"""

import numpy as np
import pytest
import torch

import oracle
import paper_2501_14577_amd as zeta
import workloads
from gpu_util import device, host, i32_to_dev, inputs, log, oracle_select, to_dev

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _lib():
    device()
    zeta.load_library()


def _close(got, ref, name):
    tol = 1e-4 * (1.0 + float(np.abs(ref).max()))
    err = float(np.abs(got - ref).max())
    assert err <= tol, (name, err, tol)


def _gpu(raw, dout_raw, w, causal, eps, chunk=0, order="level"):
    """Encode, sort, order and select on the GPU (one-pass forward, which also
    returns the windows), then the one-pass gradients.  ``order``: "level"
    (zeta_query_order), "position" (none) or a host permutation [S, N]."""
    S = raw["q"].shape[0]
    q, k, v, dout = (to_dev(a[None], w.dtype) for a in (raw["q"], raw["k"], raw["v"], dout_raw))
    res = zeta.forward(q, k, v, w.topk, eps, causal, w.bits, fused=True, chunk=chunk, return_intermediates=True)
    if isinstance(order, str):
        q_order = res["q_order"] if order == "level" else None
    else:
        q_order = i32_to_dev(order[None])
    grads = zeta.zeta_select_attend_bwd(q, k, v, res["q_codes"], res["sorted_codes"], res["perm"], w.topk, causal,
                                        eps, dout, chunk=chunk, q_order=q_order)
    torch.cuda.synchronize()
    idx = host(res["idx"]).reshape(S, w.N, w.topk)
    dq, dk, dv, deps = (host(t) for t in grads)
    return idx, dq.reshape(S, w.N, -1), dk.reshape(S, w.N, -1), dv.reshape(S, w.N, -1), float(deps[0])


def _check(idx, got, f, dout, eps):
    dq, dk, dv, deps = got
    rq, rk, rv, reps = oracle.attend_bwd(f["q"], f["k"], f["v"], idx, eps, dout)
    _close(dq, rq, "dq")
    _close(dk, rk, "dk")
    _close(dv, rv, "dv")
    assert abs(deps - reps) <= 1e-4 * (1.0 + abs(reps)), (deps, reps)


# (config, causal, segments compared)
CFGS = [(2, True, 4), (3, False, 3), (3, True, 3), (4, True, 2)]


@pytest.mark.parametrize("cfg,causal,nseg", CFGS)
def test_tile_bwd_config(cfg, causal, nseg):
    w, x, f = inputs(cfg)
    log(f"tile bwd config {cfg} causal={causal} segments={nseg}")
    S = w.segments
    raw = {n: a.reshape(S, w.N, -1)[:nseg] for n, a in x.items()}
    fs = {n: a[:nseg] for n, a in f.items()}
    dout_raw = workloads.generate_dout(w).reshape(S, w.N, w.dv)[:nseg]
    idx, *got = _gpu(raw, dout_raw, w, causal, 0.5)
    assert np.array_equal(idx, oracle_select(cfg, causal)[:nseg])
    _check(idx, got, fs, oracle.as_f32(dout_raw, w.dtype), 0.5)


EDGE = [
    dict(N=1, topk=8, dv=64),
    dict(N=37, topk=7, dv=32),
    dict(N=129, topk=1, dv=64),
    dict(N=500, topk=64, dv=128),
    dict(N=700, topk=1024, dv=256),
    dict(N=1000, topk=16, dv=32, chunk=100),
    dict(N=2000, topk=40, dv=64, chunk=256),
    # The window search's 32-bit positions (segments over 65536 rows).
    dict(N=70001, topk=16, dv=32, chunk=5000),
]


@pytest.mark.parametrize("shape", EDGE, ids=[f"N{e['N']}-k{e['topk']}-dv{e['dv']}-c{e.get('chunk', 0)}" for e in EDGE])
@pytest.mark.parametrize("causal", [False, True])
def test_tile_bwd_edges(shape, causal):
    """Small and ragged shapes (tiles past the segment's end, N below one
    tile), every d_v, k >= N, k = 1, the chunked rule (first chunk: empty
    pools) and both modes, with eps != 0.5."""
    chunk = shape.get("chunk", 0) if causal else 0
    w = workloads.custom(B=1, H=3, N=shape["N"], dv=shape["dv"], topk=shape["topk"], dtype="bf16", bits=8,
                         seed=shape["N"] * 3 + shape["topk"])
    log(f"tile bwd edge {shape} causal={causal}")
    x = workloads.generate(w)
    S = w.segments
    raw = {n: a.reshape(S, w.N, -1) for n, a in x.items()}
    f = {n: oracle.as_f32(a, w.dtype) for n, a in raw.items()}
    dout_raw = workloads.generate_dout(w).reshape(S, w.N, w.dv)
    idx, *got = _gpu(raw, dout_raw, w, causal, 0.3, chunk=chunk)
    qc, kc, _, _ = oracle.morton_encode(f["q"], f["k"], w.bits)
    assert np.array_equal(idx, oracle.select_topk(qc, kc, w.topk, causal, chunk=chunk))
    _check(idx, got, f, oracle.as_f32(dout_raw, w.dtype), 0.3)


@pytest.mark.parametrize("N", [4096, 4097, 16385, 65537, 131073])
def test_tile_bwd_tile_counts(N):
    """Segments around the tile counts (N / 16) at which the candidate ranges
    of the key pass change kernels, the last in memory, with deps summed from
    ragged last tiles."""
    w = workloads.custom(B=1, H=1, N=N, dv=32, topk=8, dtype="bf16", bits=8, seed=N)
    log(f"tile bwd tile counts N={N}")
    x = workloads.generate(w)
    raw = {n: a.reshape(1, N, -1) for n, a in x.items()}
    f = {n: oracle.as_f32(a, w.dtype) for n, a in raw.items()}
    dout_raw = workloads.generate_dout(w).reshape(1, N, w.dv)
    idx, *got = _gpu(raw, dout_raw, w, True, 0.5)
    _check(idx, got, f, oracle.as_f32(dout_raw, w.dtype), 0.5)


@pytest.mark.parametrize("N,topk", [(4200, 100), (8300, 160), (8300, 300), (8300, 512)])
@pytest.mark.parametrize("chunk", [0, 70])
def test_tile_bwd_first_lists(N, topk, chunk):
    """The gradients' first prefix list serves queries with few keys in their
    pool, down to one: it starts two levels later than the forward's (k = 100),
    one (160), or at the same (300, 512: a longer list would not be staged
    whole)."""
    w = workloads.custom(B=1, H=2, N=N, dv=32, topk=topk, dtype="bf16", bits=8, seed=topk)
    log(f"tile bwd first lists N={N} k={topk} chunk={chunk}")
    raw = {n: a.reshape(2, N, -1) for n, a in workloads.generate(w).items()}
    f = {n: oracle.as_f32(a, w.dtype) for n, a in raw.items()}
    dout_raw = workloads.generate_dout(w).reshape(2, N, w.dv)
    idx, *got = _gpu(raw, dout_raw, w, True, 0.5, chunk=chunk)
    _check(idx, got, f, oracle.as_f32(dout_raw, w.dtype), 0.5)


@pytest.mark.parametrize("dv", [32, 128])
def test_tile_bwd_nan_without_window(dv):
    """The chunked rule leaves the first chunk's queries without a window:
    whatever their dout rows hold (here NaN and infinities, the first row's
    among them), no gradient changes, also where an order mixes them and
    several lists in one tile."""
    w = workloads.custom(B=1, H=2, N=1000, dv=dv, topk=16, dtype="bf16", bits=8, seed=dv)
    log(f"tile bwd NaN dout without window dv={dv}")
    raw = {n: a.reshape(2, w.N, -1) for n, a in workloads.generate(w).items()}
    clean = workloads.generate_dout(w).reshape(2, w.N, dv).copy()
    clean[:, :100] = 0
    dirty = clean.copy()
    dirty[:, :100:3] = np.array(0x7FC0).astype(dirty.dtype)
    dirty[:, 1:100:3] = np.array(0x7F80).astype(dirty.dtype)
    rng = np.random.default_rng(dv)
    perm = np.stack([rng.permutation(w.N) for _ in range(2)]).astype(np.int32)
    for order in ("level", "position", perm):
        want = _gpu(raw, clean, w, True, 0.5, chunk=100, order=order)
        got = _gpu(raw, dirty, w, True, 0.5, chunk=100, order=order)
        for a, b in zip(got, want):
            assert np.array_equal(a, b)


@pytest.mark.parametrize("what", ["dout", "q"])
@pytest.mark.parametrize("dv", [64, 128])
def test_tile_bwd_nonfinite_row_stays_in_its_window(dv, what):
    """A NaN or infinite dout (or q) row of a query reaches the keys of its
    window and no others: every other key has the gradients it has with that
    row finite, to rounding (sums that meet such a row are formed in another
    way).  Enough rows that a wavefront of the key pass takes two chunks, an
    odd number of them."""
    w = workloads.custom(B=1, H=8, N=4112, dv=dv, topk=16, dtype="bf16", bits=8, seed=dv + 5)
    log(f"tile bwd non-finite {what} row dv={dv}")
    S, N = w.segments, w.N
    q, k, v = (to_dev(a.reshape(1, S, N, -1), w.dtype) for a in workloads.generate(w).values())
    res = zeta.forward(q, k, v, w.topk, 0.5, False, w.bits, fused=True, return_intermediates=True)
    idx = host(res["idx"]).reshape(S, N, w.topk)
    seg = np.arange(S)
    dirty_q = np.random.default_rng(dv).integers(0, N, S)
    dout = to_dev(workloads.generate_dout(w).reshape(1, S, N, dv), w.dtype)
    dout[0, seg, dirty_q] = 0

    def grads():
        g = zeta.zeta_select_attend_bwd(q, k, v, res["q_codes"], res["sorted_codes"], res["perm"], w.topk, False, 0.5,
                                        dout, q_order=res["q_order"])
        torch.cuda.synchronize()
        return [host(t).reshape(S, N, -1) for t in g[:3]]

    _, ck, cv = grads()
    bad = torch.tensor([float("inf"), float("nan")] * (S // 2), dtype=torch.bfloat16, device=q.device)
    (dout if what == "dout" else q)[0, seg, dirty_q] = bad[:, None]
    _, gk, gv = grads()
    for s in range(S):
        away = np.setdiff1d(np.arange(N), idx[s, dirty_q[s]])
        _close(gk[s, away], ck[s, away], f"dk {s}")
        _close(gv[s, away], cv[s, away], f"dv {s}")
        assert not np.isfinite((gv if what == "dout" else gk)[s, idx[s, dirty_q[s]]]).any()


@pytest.mark.parametrize("what", ["v", "k"])
@pytest.mark.parametrize("N,H,order", [(4112, 8, "level"), (1000, 2, "level"), (1000, 2, "random")])
def test_tile_bwd_nonfinite_key_stays_with_its_queries(N, H, order, what):
    """NaN and infinite rows of v (or k) reach the queries whose windows hold
    them and the other keys of those windows; every other query's dq has the
    bits and every other key's dk and dv the values to rounding that they have
    with those rows finite, whatever lists, chunks and tiles they share with
    them, and the dk and dv of a key in no window stay zero."""
    w = workloads.custom(B=1, H=H, N=N, dv=64, topk=16, dtype="bf16", bits=8, seed=N + 9)
    log(f"tile bwd non-finite {what} rows N={N} order={order}")
    rng = np.random.default_rng(N)
    q, k, v = (to_dev(a.reshape(1, H, N, -1), w.dtype) for a in workloads.generate(w).values())
    q *= 0.3  # leaves keys in no window
    dout = to_dev(workloads.generate_dout(w).reshape(1, H, N, 64), w.dtype)
    res = zeta.forward(q, k, v, w.topk, 0.5, True, w.bits, fused=True, return_intermediates=True)
    idx = host(res["idx"]).reshape(H, N, w.topk)
    given = res["q_order"] if order == "level" else i32_to_dev(
        np.stack([rng.permutation(N) for _ in range(H)])[None].astype(np.int32))

    def grads():
        g = zeta.zeta_select_attend_bwd(q, k, v, res["q_codes"], res["sorted_codes"], res["perm"], w.topk, True, 0.5,
                                        dout, q_order=given)
        torch.cuda.synchronize()
        return [host(t).reshape(H, N, -1) for t in g[:3]]

    clean = grads()
    bad = np.zeros((H, N), bool)
    for s in range(H):
        used = np.unique(idx[s])
        bad[s, rng.choice(np.setdiff1d(np.arange(N), used), 6, replace=False)] = True
        bad[s, rng.choice(used[used >= 0], 6, replace=False)] = True
    value = np.where(rng.random((H, N)) < 0.5, np.inf, np.nan)[bad]
    (v if what == "v" else k)[0][torch.from_numpy(bad).to(q.device)] = to_dev(value, "f32").to(torch.bfloat16)[:, None]
    dirty = grads()
    for s in range(H):
        holds = (bad[s][idx[s]] & (idx[s] >= 0)).any(1)
        spoiled = np.unique(idx[s][holds])
        keys = np.setdiff1d(np.arange(N), spoiled)
        assert holds.any() and bad[s, keys].any()
        assert np.array_equal(dirty[0][s, ~holds], clean[0][s, ~holds]), s
        for t in (1, 2):
            _close(dirty[t][s, keys], clean[t][s, keys], f"{s} {t}")
            assert not dirty[t][s, np.setdiff1d(np.arange(N), idx[s])].any()


@pytest.mark.parametrize("N,H,dv", [(1000, 2, 32), (4112, 8, 64)])
def test_tile_bwd_nonfinite_rows_of_early_queries(N, H, dv):
    """Non-finite dout rows of queries among the first 60 positions reach no
    key from position 60 on and no other query, also where an order mixes
    queries of several lists in one tile and where their list holds later
    keys."""
    w = workloads.custom(B=1, H=H, N=N, dv=dv, topk=16, dtype="bf16", bits=8, seed=dv + 6)
    log(f"tile bwd non-finite dout row of another list N={N} dv={dv}")
    raw = {n: a.reshape(H, N, -1) for n, a in workloads.generate(w).items()}
    clean = workloads.generate_dout(w).reshape(H, N, dv).copy()
    clean[:, 3:60:7] = 0
    dirty = clean.copy()
    dirty[:, 3:60:14] = np.array(0x7FC0).astype(dirty.dtype)
    dirty[:, 10:60:14] = np.array(0x7F80).astype(dirty.dtype)
    others = np.setdiff1d(np.arange(N), np.arange(3, 60, 7))
    rng = np.random.default_rng(N)
    perm = np.stack([rng.permutation(N) for _ in range(H)]).astype(np.int32)
    for order in ("level", "position", perm):
        _, cq, ck, cv, _ = _gpu(raw, clean, w, True, 0.5, order=order)
        _, gq, gk, gv, _ = _gpu(raw, dirty, w, True, 0.5, order=order)
        assert np.array_equal(gq[:, others], cq[:, others])
        _close(gk[:, 60:], ck[:, 60:], "dk")
        _close(gv[:, 60:], cv[:, 60:], "dv")


def test_tile_bwd_orders_and_repeat():
    """Any processing order gives the oracle's gradients; dq and deps's parts
    depend only on each query's own window, so dq is bit-identical across
    orders; a repeated call gives the same bits for every output."""
    cfg = 2
    w, x, f = inputs(cfg)
    log("tile bwd processing orders")
    S = 4
    raw = {n: a.reshape(w.segments, w.N, -1)[:S] for n, a in x.items()}
    fs = {n: a[:S] for n, a in f.items()}
    dout_raw = workloads.generate_dout(w).reshape(w.segments, w.N, w.dv)[:S]
    dout = oracle.as_f32(dout_raw, w.dtype)
    rng = np.random.default_rng(9)
    perm = np.stack([rng.permutation(w.N) for _ in range(S)]).astype(np.int32)
    runs = {o if isinstance(o, str) else "random": _gpu(raw, dout_raw, w, True, 0.5, order=o)
            for o in ("level", "position", perm)}
    for name, (idx, *got) in runs.items():
        _check(idx, got, fs, dout, 0.5)
    assert np.array_equal(runs["level"][1], runs["position"][1])
    assert np.array_equal(runs["level"][1], runs["random"][1])
    again = _gpu(raw, dout_raw, w, True, 0.5)
    for t in range(1, 5):
        assert np.array_equal(np.asarray(runs["level"][t]), np.asarray(again[t])), t


@pytest.mark.parametrize("order", ["level", "position", "random"])
@pytest.mark.parametrize("dv,N,causal", [(64, 8200, True), (64, 8200, False), (128, 4113, True)])
def test_tile_bwd_two_chunks(dv, N, causal, order):
    """Enough rows that a wavefront of the key pass takes two chunks of the
    long lists and one of the short ones, an odd number of chunks, at the value
    widths the workloads train with, in each kind of processing order."""
    w = workloads.custom(B=1, H=8, N=N, dv=dv, topk=32, dtype="bf16", bits=10, seed=dv + N)
    log(f"tile bwd two chunks dv={dv} N={N} causal={causal} order={order}")
    raw = {n: a.reshape(8, N, -1) for n, a in workloads.generate(w).items()}
    f = {n: oracle.as_f32(a, w.dtype) for n, a in raw.items()}
    dout_raw = workloads.generate_dout(w).reshape(8, N, dv)
    rng = np.random.default_rng(N)
    given = np.stack([rng.permutation(N) for _ in range(8)]).astype(np.int32) if order == "random" else order
    idx, *got = _gpu(raw, dout_raw, w, causal, 0.5, order=given)
    _check(idx, got, f, oracle.as_f32(dout_raw, w.dtype), 0.5)


def test_tile_bwd_deps_many_tiles():
    """deps over more than 131072 tiles (summed in two stages), with values and
    upstream gradients that give every query's part the same sign: dout_i . v_j
    falls with |q_i - k_j|^2, so a missing or repeated part shows.  The
    reference sums the definition in float64 over the same windows."""
    B, H, N, dv, topk = 1, 2100, 1024, 32, 4
    log(f"tile bwd deps over {H * N // 16} tiles")
    g = torch.Generator(device=device()).manual_seed(3)
    q, k = (torch.randn((B, H, N, 3), generator=g, device=device()).to(torch.bfloat16) for _ in range(2))
    v, dout = (torch.zeros((B, H, N, dv), dtype=torch.bfloat16, device=device()) for _ in range(2))
    v[..., :3], v[..., 3], v[..., 4] = k, -0.5 * k.float().square().sum(-1), 1
    dout[..., :3], dout[..., 3], dout[..., 4] = q, 1, -0.5 * q.float().square().sum(-1)
    res = zeta.forward(q, k, v, topk, 0.5, False, 10, fused=True, return_intermediates=True)
    deps = zeta.zeta_select_attend_bwd(q, k, v, res["q_codes"], res["sorted_codes"], res["perm"], topk, False, 0.5, dout,
                                       q_order=res["q_order"])[3]
    ref, parts = 0.0, []
    for s in range(0, H, 300):
        Q, K, V, D = (t[0, s:s + 300].double() for t in (q, k, v, dout))
        at = res["idx"][0, s:s + 300].long().reshape(len(Q), -1, 1)
        Kj, Vj = (t.gather(1, at.expand(-1, -1, t.shape[-1])).view(len(Q), N, topk, -1) for t in (K, V))
        S = 1 / ((Q[:, :, None] - Kj).square().sum(-1) + 0.5)
        Z = S.sum(-1, keepdim=True)
        p = (Vj * D[:, :, None]).sum(-1)
        part = -((p - (S / Z * p).sum(-1, keepdim=True)) * S.square() / Z).sum(-1)
        parts.append(float((part > 0).double().mean()))
        ref += float(part.sum())
    assert max(parts) < 0.01, "all but a few parts are negative"
    assert abs(float(deps[0]) - ref) <= 1e-4 * (1.0 + abs(ref)), (float(deps[0]), ref)


def test_tile_bwd_long_context():
    """The long-context workload at full size, as the benchmark runs it: every
    gradient matches zeta_topk_attn_bwd (the per-query path, pinned to the
    oracle above) on the same windows, and the invariants of the definition
    hold (sum dq + sum dk = 0 per segment, sum dv = sum dout)."""
    cfg = 5
    w, x, _ = inputs(cfg)
    log("tile bwd long context")
    S = w.segments
    raw = {n: a.reshape(S, w.N, -1) for n, a in x.items()}
    dout_raw = workloads.generate_dout(w).reshape(S, w.N, w.dv)
    q, k, v, dout = (to_dev(a[None], w.dtype) for a in (raw["q"], raw["k"], raw["v"], dout_raw))
    res = zeta.forward(q, k, v, w.topk, 0.5, True, w.bits, return_intermediates=True)
    ref = zeta.zeta_topk_attn_bwd(q, k, v, res["idx"], dout, 0.5, q_order=res["q_order"])
    got = zeta.zeta_select_attend_bwd(q, k, v, res["q_codes"], res["sorted_codes"], res["perm"], w.topk, True, 0.5,
                                      dout, q_order=res["q_order"])
    torch.cuda.synchronize()
    names = ("dq", "dk", "dv", "deps")
    for name, a, b in zip(names, got, ref):
        a, b = host(a).astype(np.float64), host(b).astype(np.float64)
        if name == "deps":
            assert abs(a[0] - b[0]) <= 1e-4 * (1.0 + abs(b[0])), (a, b)
        else:
            _close(a, b, name)
    dq, dk, dv = (host(t).reshape(S, w.N, -1).astype(np.float64) for t in got[:3])
    dsum = dq.sum(axis=1) + dk.sum(axis=1)
    scale = np.abs(dq).sum(axis=1) + np.abs(dk).sum(axis=1)
    assert np.all(np.abs(dsum) <= 1e-4 * (1.0 + scale)), (dsum, scale)
    dsv = oracle.as_f32(dout_raw, w.dtype).astype(np.float64).sum(axis=1)
    assert np.allclose(dv.sum(axis=1), dsv, rtol=1e-4, atol=1e-2), np.abs(dv.sum(axis=1) - dsv).max()


HIST = [(2, True, 2), (3, False, 2), (3, True, 2)]


@pytest.mark.parametrize("cfg,causal,nseg", HIST)
def test_tile_bwd_history(cfg, causal, nseg):
    """With the history-mean candidate (means from zeta_history_mean, the
    same causal flag): the one-pass gradients match the oracle's, whose means
    and gradients through them are its own (Section 3.4)."""
    w, x, f = inputs(cfg)
    log(f"tile bwd history config {cfg} causal={causal}")
    S = w.segments
    raw = {n: a.reshape(S, w.N, -1)[:nseg] for n, a in x.items()}
    fs = {n: a[:nseg] for n, a in f.items()}
    dout_raw = workloads.generate_dout(w).reshape(S, w.N, w.dv)[:nseg]
    q, k, v, dout = (to_dev(a[None], w.dtype) for a in (raw["q"], raw["k"], raw["v"], dout_raw))
    res = zeta.forward(q, k, v, w.topk, 0.5, causal, w.bits, fused=True, history=True, return_intermediates=True)
    grads = zeta.zeta_select_attend_bwd(q, k, v, res["q_codes"], res["sorted_codes"], res["perm"], w.topk, causal,
                                        0.5, dout, q_order=res["q_order"], mean_k=res["mean_k"], mean_v=res["mean_v"])
    torch.cuda.synchronize()
    idx = host(res["idx"]).reshape(nseg, w.N, w.topk)
    dq, dk, dv, deps = (host(t) for t in grads)
    rq, rk, rv, reps = oracle.attend_bwd(fs["q"], fs["k"], fs["v"], idx, 0.5, oracle.as_f32(dout_raw, w.dtype),
                                         history=True, causal=causal)
    _close(dq.reshape(rq.shape), rq, "dq")
    _close(dk.reshape(rk.shape), rk, "dk")
    _close(dv.reshape(rv.shape), rv, "dv")
    assert abs(float(deps[0]) - reps) <= 1e-4 * (1.0 + abs(reps)), (float(deps[0]), reps)


@pytest.mark.parametrize("dv", [32, 128, 256])
@pytest.mark.parametrize("causal", [True, False])
def test_tile_bwd_history_widths(dv, causal):
    """The one-pass gradients with the history-mean candidate at the value
    widths the configurations do not use, on a ragged length, both modes."""
    w = workloads.custom(B=1, H=2, N=650, dv=dv, topk=24, dtype="bf16", bits=8, seed=dv + 11)
    log(f"tile bwd history dv={dv} causal={causal}")
    x = workloads.generate(w)
    S = w.segments
    raw = {n: a.reshape(S, w.N, -1) for n, a in x.items()}
    f = {n: oracle.as_f32(a, w.dtype) for n, a in raw.items()}
    dout_raw = workloads.generate_dout(w).reshape(S, w.N, w.dv)
    q, k, v, dout = (to_dev(a[None], w.dtype) for a in (raw["q"], raw["k"], raw["v"], dout_raw))
    res = zeta.forward(q, k, v, w.topk, 0.5, causal, w.bits, fused=True, history=True, return_intermediates=True)
    grads = zeta.zeta_select_attend_bwd(q, k, v, res["q_codes"], res["sorted_codes"], res["perm"], w.topk, causal,
                                        0.5, dout, q_order=res["q_order"], mean_k=res["mean_k"], mean_v=res["mean_v"])
    torch.cuda.synchronize()
    idx = host(res["idx"]).reshape(S, w.N, w.topk)
    dq, dk, dv_, deps = (host(t) for t in grads)
    rq, rk, rv, reps = oracle.attend_bwd(f["q"], f["k"], f["v"], idx, 0.5, oracle.as_f32(dout_raw, w.dtype),
                                         history=True, causal=causal)
    _close(dq.reshape(rq.shape), rq, "dq")
    _close(dk.reshape(rk.shape), rk, "dk")
    _close(dv_.reshape(rv.shape), rv, "dv")
    assert abs(float(deps[0]) - reps) <= 1e-4 * (1.0 + abs(reps)), (float(deps[0]), reps)


def test_tile_bwd_history_two_chunks():
    """The history-mean candidate where a wavefront of the key pass takes two
    chunks (d_v = 64, 8 segments of 8200 rows)."""
    N, topk = 8200, 32
    w = workloads.custom(B=1, H=8, N=N, dv=64, topk=topk, dtype="bf16", bits=10, seed=77)
    log("tile bwd history two chunks")
    raw = {n: a.reshape(8, N, -1) for n, a in workloads.generate(w).items()}
    f = {n: oracle.as_f32(a, w.dtype) for n, a in raw.items()}
    dout_raw = workloads.generate_dout(w).reshape(8, N, 64)
    q, k, v, dout = (to_dev(a[None], w.dtype) for a in (raw["q"], raw["k"], raw["v"], dout_raw))
    res = zeta.forward(q, k, v, topk, 0.5, True, w.bits, fused=True, history=True, return_intermediates=True)
    grads = zeta.zeta_select_attend_bwd(q, k, v, res["q_codes"], res["sorted_codes"], res["perm"], topk, True, 0.5, dout,
                                        q_order=res["q_order"], mean_k=res["mean_k"], mean_v=res["mean_v"])
    torch.cuda.synchronize()
    idx = host(res["idx"]).reshape(8, N, topk)
    want = oracle.attend_bwd(f["q"], f["k"], f["v"], idx, 0.5, oracle.as_f32(dout_raw, w.dtype), history=True, causal=True)
    for name, got, ref in zip(("dq", "dk", "dv"), grads, want):
        _close(host(got).reshape(ref.shape), ref, name)
    assert abs(float(grads[3][0]) - want[3]) <= 1e-4 * (1.0 + abs(want[3])), (float(grads[3][0]), want[3])


@pytest.mark.parametrize("N,topk,dv,causal,history", [(1, 1, 32, True, False), (1000, 16, 64, True, False), (4113, 100, 128, True, True),
                                                      (4113, 100, 32, False, True), (700, 1024, 256, True, False),
                                                      (131073, 8, 32, True, False)])
def test_tile_bwd_workspace_bound(N, topk, dv, causal, history):
    """The call stays within the size it asks for, and its results do not
    depend on what the buffer held."""
    w = workloads.custom(B=1, H=2, N=N, dv=dv, topk=topk, dtype="bf16", bits=8, seed=N)
    log(f"tile bwd workspace bound N={N} k={topk} dv={dv} causal={causal} history={history}")
    q, k, v = (to_dev(a.reshape(1, 2, N, -1), w.dtype) for a in workloads.generate(w).values())
    dout = to_dev(workloads.generate_dout(w).reshape(1, 2, N, dv), w.dtype)
    res = zeta.forward(q, k, v, topk, 0.5, causal, w.bits, fused=True, history=history, return_intermediates=True)
    n = zeta.zeta_select_attend_bwd_workspace_size(1, 2, N, dv, topk, causal, history)
    runs = []
    for fill in (0x00, 0xFF):
        buf = torch.full((n + 8192,), fill, dtype=torch.uint8, device=device())
        g = zeta.zeta_select_attend_bwd(q, k, v, res["q_codes"], res["sorted_codes"], res["perm"], topk, causal, 0.5, dout,
                                        q_order=res["q_order"], mean_k=res["mean_k"], mean_v=res["mean_v"],
                                        workspace=buf[:n])
        torch.cuda.synchronize()
        assert bool((buf[n:] == fill).all())
        runs.append([host(t) for t in g])
    for a, b in zip(*runs):
        assert np.array_equal(a, b) and np.isfinite(a).all()
