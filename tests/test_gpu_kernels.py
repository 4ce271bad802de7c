"""Kernel-level parity on the GPU against the CPU oracle, through the C ABI's
kernel entry points (device buffers allocated with torch).

Tolerances follow from the kernels' arithmetic (u = 2^-11, the f16 unit
roundoff):
 * GEMM: weights d * (q - 8) rounded to f16 (<= u relative) on f16 activations
   (exact inputs), fp32 accumulation: |y - y_ref| <= 2u * sum_k |x_k w_k|
   (+ u |y| for the f16 SwiGLU output).
 * Attention: scores in fp32 from f16 operands (exact products), P rounded to
   f16 (<= u relative), output rounded to f16: |o - o_ref| <= 2u |o_ref| +
   2u max|v|.
 * RMSNorm: fp32 sum of squares, f16 output: 2u relative.
"""

import numpy as np
import pytest

import oracle as O
from paper_2609_01338_amd import mz
from paper_2609_01338_amd import workloads as W
from gpu_util import F16_REL, report, stream, torch_cuda

REL = 2 * F16_REL

pytestmark = pytest.mark.gpu


def _gemm_case(M, N, K, epi, seed, sample_rows=None, n_split=None):
    """n_split: None for mz_q4_gemm, "queued" for mz_q4_gemm_queued (run
    twice from the same initial output on the same queues, which must come
    back zero, and equal to mz_q4_gemm bit for bit), "long-k" for
    mz_q4_gemm_ex with the restore's 64 MiB workspace on a shape it splits
    over K as 256-row tiles, else mz_q4_gemm_split with that many K splits
    ("auto": the restore's choice)."""
    torch = torch_cuda()
    rng = np.random.default_rng(seed)
    report("gemm", M=M, N=N, K=K, epi=epi, seed=seed, n_split=n_split)
    if sample_rows is not None:   # checked on the host: the gather below must stay in bounds
        assert 0 <= int(np.min(sample_rows)) and int(np.max(sample_rows)) < M, "sample rows out of range"
    if epi == 2:
        g = W.encode_q4_0((rng.standard_normal((N, K)) * 0.02).astype(np.float32))
        u = W.encode_q4_0((rng.standard_normal((N, K)) * 0.02).astype(np.float32))
        packed = mz.mz_q4_gemm_pack(g, N, K, w_up=u)
        n_pad = 2 * ((N + 127) // 128 * 128)
    else:
        raw = W.encode_q4_0((rng.standard_normal((N, K)) * 0.02).astype(np.float32))
        packed = mz.mz_q4_gemm_pack(raw, N, K)
        n_pad = (N + 255) // 256 * 256
    gen = torch.Generator(device="cuda").manual_seed(seed)
    x = torch.randn(M, K, device="cuda", generator=gen).to(torch.float16)
    w = torch.from_numpy(packed).cuda()
    if epi == 2:
        y = torch.zeros(M, n_pad // 2, device="cuda", dtype=torch.float16)
    else:
        y = torch.randn(M, n_pad, device="cuda", generator=gen) if epi == 1 else \
            torch.zeros(M, n_pad, device="cuda")
    y0 = y.float().cpu().numpy().astype(np.float64)
    if n_split is None:
        mz.mz_q4_gemm(x.data_ptr(), M, n_pad, K, w.data_ptr(), epi, y.data_ptr(), stream())
    elif n_split == "queued":
        y_init = y.clone()
        mz.mz_q4_gemm(x.data_ptr(), M, n_pad, K, w.data_ptr(), epi, y.data_ptr(), stream())
        plain = y.clone()
        queues = torch.zeros(16, device="cuda", dtype=torch.int32)
        for rep in range(2):
            y.copy_(y_init)
            mz.mz_q4_gemm_queued(x.data_ptr(), M, n_pad, K, w.data_ptr(), epi, y.data_ptr(), queues.data_ptr(),
                                 stream())
            torch.cuda.synchronize()
            assert int(queues.abs().sum()) == 0, "work queues not left at zero"
            assert torch.equal(y.view(torch.uint8), plain.view(torch.uint8)), "queued != mz_q4_gemm"
    elif n_split in ("long-k", "workspace"):
        wsb = 64 << 20
        report("  plan", plan=mz.mz_q4_gemm_plan(M, n_pad, K, wsb))
        if n_split == "long-k":
            assert mz.mz_q4_gemm_long_k_splits(M, n_pad, K, wsb) > 1, "shape outside the long-K split rule"
        ws = torch.full((wsb // 4,), float("nan"), device="cuda")      # stale partials must not leak in
        mz.mz_q4_gemm_ex(x.data_ptr(), M, n_pad, K, w.data_ptr(), epi, y.data_ptr(), stream(),
                         workspace=ws.data_ptr(), workspace_bytes=wsb)
    else:
        if n_split == "auto":
            n_split = mz.mz_q4_gemm_auto_splits(M, n_pad, K, 64 << 20)
            report("  auto splits", n_split=n_split)
        wsb = mz.mz_q4_gemm_split_workspace_bytes(M, n_pad, n_split)
        ws = torch.full((wsb // 4,), float("nan"), device="cuda")      # stale partials must not leak in
        mz.mz_q4_gemm_split(x.data_ptr(), M, n_pad, K, w.data_ptr(), epi, y.data_ptr(), n_split, ws.data_ptr(),
                            wsb, stream())
    torch.cuda.synchronize()
    rows = np.arange(M) if sample_rows is None else sample_rows
    xs = x[torch.from_numpy(rows).cuda()].float().cpu().numpy().astype(np.float64)
    ys = y.float().cpu().numpy()[rows].astype(np.float64)
    if epi == 2:
        G = O.q4_0_decode(g.reshape(-1), N, K)
        U = O.q4_0_decode(u.reshape(-1), N, K)
        gr, ur = xs @ G.T, xs @ U.T
        bg = REL * (np.abs(xs) @ np.abs(G).T) + 1e-6
        bu = REL * (np.abs(xs) @ np.abs(U).T) + 1e-6
        ref = O.silu(gr) * ur
        bound = 1.1 * bg * (np.abs(ur) + bu) + np.abs(O.silu(gr)) * bu + REL * np.abs(ref) + 1e-6
        got = ys[:, :N]
        assert np.all(ys[:, N:] == 0)          # padded gate/up columns give silu(0) * 0
    else:
        Wd = O.q4_0_decode(raw.reshape(-1), N, K)
        ref = xs @ Wd.T + (y0[rows, :N] if epi == 1 else 0.0)
        bound = REL * (np.abs(xs) @ np.abs(Wd).T) + 1e-5 * (1 + np.abs(ref))
        got = ys[:, :N]
    err = np.abs(got - ref)
    report("  err", max=float(err.max()), worst_ratio=float((err / bound).max()))
    assert np.all(err <= bound)


@pytest.mark.parametrize("M,N,K,epi", [
    (1, 128, 64, 0), (200, 256, 128, 0), (333, 512, 704, 0), (129, 384, 256, 1),
    (77, 688, 256, 2), (300, 1408, 256, 2)])
def test_gemm_small(M, N, K, epi):
    _gemm_case(M, N, K, epi, seed=M + N + K)


@pytest.mark.parametrize("M,N,K,epi", [
    (1, 256, 640, 0), (5, 512, 1024, 1), (64, 384, 960, 2), (129, 1024, 4096, 1), (200, 688, 512, 2),
    (1, 1408, 2048, 2), (33, 256, 4096, 0)])
def test_gemm_split(M, N, K, epi):
    """Split-K against the exact product: splits that divide the K steps,
    ragged last splits, one step per split, and the restore's choice."""
    nk = K // 64
    for ns in sorted({2, 3, nk, "auto"} - {1}, key=str):
        if ns != "auto" and ns > nk:
            continue
        _gemm_case(M, N, K, epi, seed=M + N + K, n_split=ns)


@pytest.mark.parametrize("M,N,K,epi", [(2048, 2048, 8192, 1), (2000, 2048, 8192, 0), (2048, 2048, 4096, 0),
                                       (2048, 1024, 8192, 2)])
def test_gemm_long_k_split(M, N, K, epi):
    """Products with too few 256-row tiles for the chip but a long K range,
    as the restore launches them (with its workspace): 128 x 128 tiles in two
    splits, of half the K range in one.  The 1B down projection, a ragged last
    row tile, half the K range, and the SwiGLU epilogue, against the exact
    product on one row in every 64-row tile."""
    plan = [p[1:] for p in mz.mz_q4_gemm_plan(M, 2 * N if epi == 2 else N, K, 64 << 20)]
    assert plan == [(128, 128, 2 if K == 8192 else 1)]
    _gemm_case(M, N, K, epi, seed=M + N + K + 5, sample_rows=_tile_rows(M, 64, M + K), n_split="long-k")


@pytest.mark.parametrize("M,plan", [(17, (32, 128, 16)), (40, (64, 128, 8)), (128, (128, 128, 8)), (1000, (128, 256, 4)),
                                    (1900, (128, 256, 2)), (1921, (256, 256, 2)), (2048, (256, 256, 2))])
def test_gemm_planned_splits(M, plan):
    """The 8B down projection as the restore launches it (64 MiB of workspace,
    NaN before the call) in every tile form that splits over K, against the
    exact product on one row in every 64-row tile; the plan says which form
    runs."""
    N, K = 4096, 14336
    assert mz.mz_q4_gemm_plan(M, N, K, 64 << 20) == [(M, *plan)]
    _gemm_case(M, N, K, 1, seed=M, sample_rows=_tile_rows(M, 64, M), n_split="workspace")


@pytest.mark.parametrize("m,N,K", [(2, 512, 704), (17, 1024, 2048), (200, 768, 1088), (1500, 512, 1024)])
def test_gemm_split_count_kept(m, N, K):
    """A split count other than mz_q4_gemm_auto_splits' own is taken as it is:
    the ranges of ceil(steps / n_split) steps, each the bits of mz_q4_gemm on
    its part of K, added in order in fp32.  Down to one step per range,
    trailing empty ranges and one range among them."""
    torch = torch_cuda()
    nk = K // 64
    gen = torch.Generator(device="cuda").manual_seed(m)
    X = torch.randn(m, K, device="cuda", generator=gen).half()
    W_ = torch.randint(0, 256, (N // 256, nk, 9216), device="cuda", dtype=torch.uint8, generator=gen)
    sc = (torch.rand(N // 256, nk, 512, device="cuda", generator=gen) * 0.01 + 0.01).half()
    W_[..., 8192:] = sc.view(torch.uint8).view(N // 256, nk, 1024)
    auto = mz.mz_q4_gemm_auto_splits(m, N, K, 64 << 20)
    for n_split in sorted({1, 2, 3, 5, nk - 1, nk, nk + 5} - {auto}):
        report("split count", m=m, N=N, K=K, n_split=n_split)
        y = torch.zeros(m, N, device="cuda")
        wsb = mz.mz_q4_gemm_split_workspace_bytes(m, N, n_split)
        ws = torch.full((wsb // 4,), float("nan"), device="cuda")
        mz.mz_q4_gemm_split(X.data_ptr(), m, N, K, W_.data_ptr(), 0, y.data_ptr(), n_split, ws.data_ptr(), wsb,
                            stream())
        ref = None
        steps = (nk + n_split - 1) // n_split
        for k0 in range(0, nk, steps):
            k1 = min(k0 + steps, nk)
            xs, wp = X[:, k0 * 64:k1 * 64].contiguous(), W_[:, k0:k1].contiguous()
            part = torch.zeros(m, N, device="cuda")
            mz.mz_q4_gemm(xs.data_ptr(), m, N, (k1 - k0) * 64, wp.data_ptr(), 0, part.data_ptr(), stream())
            torch.cuda.synchronize()
            ref = part if ref is None else ref + part
        assert bool((ref != 0).any()) and torch.equal(y, ref), n_split


@pytest.mark.parametrize("M", [1, 129])
def test_gemm_split_8b_layer(M):
    """The 8B projections at a decode step (1 row) and a 128-token prompt
    (129 rows), with the restore's split choice."""
    m = W.WORKLOADS["8b"].model
    ffp = (m.d_ffn + 127) // 128 * 128
    for i, (N, K, epi) in enumerate([(m.dq, m.d_model, 0), (2 * m.dkv, m.d_model, 0), (m.d_model, m.dq, 1),
                                     (m.d_ffn, m.d_model, 2), (m.d_model, ffp, 1)]):
        _gemm_case(M, N, K, epi, seed=300 + i, n_split="auto")


def test_gemm_split_validation():
    torch_cuda()
    with pytest.raises(mz.MzError):
        mz.mz_q4_gemm_split(1, 4, 256, 640, 1, 0, 1, 2, 1, 100, None)     # workspace too small
    with pytest.raises(mz.MzError):
        mz.mz_q4_gemm_split(1, 4, 256, 640, 1, 0, 1, 0, 1, 1 << 20, None)  # n_split 0
    with pytest.raises(mz.MzError):
        mz.mz_q4_gemm_queued(1, 4, 256, 640, 1, 0, 1, 0, None)            # no work queues
    assert mz.mz_q4_gemm_auto_splits(32896, 4096, 4096, 64 << 20) == 1
    assert mz.mz_q4_gemm_auto_splits(1, 4096, 14336, 64 << 20) > 8


def _layer_gemms(key):
    w = W.WORKLOADS[key]
    m = w.model
    M = w.n_ctx + w.n_prompt
    ffp = (m.d_ffn + 127) // 128 * 128
    return [(M, m.dq + 2 * m.dkv, m.d_model, 0), (M, m.d_model, m.dq, 1),
            (M, m.d_ffn, m.d_model, 2), (M, m.d_model, ffp, 1)]


def _tile_rows(M, tile, seed):
    """One row in every `tile`-row tile (at a seeded offset inside it), the
    first and last rows, and both sides of the last whole 256-row tile."""
    rng = np.random.default_rng(seed)
    starts = np.arange(0, M, tile)
    rows = np.minimum(starts + rng.integers(0, tile, starts.size), M - 1)
    edge = [r for r in (M // 256 * 256 - 1, M // 256 * 256) if 0 <= r < M]
    return np.unique(np.concatenate([rows, [0, M - 1], edge])).astype(np.int64)


@pytest.mark.parametrize("key", ["tiny", "1b", "3b", "1p5b", "8b"])
def test_gemm_full_layer_shapes(key):
    """Every projection of the workload at its full row count, checked on one
    row in every 64-row tile (so in every tile but the 32-row ones) including
    the ragged tail and both sides of the row where whole 256-row tiles end;
    work queues passed as the restore does (a launch takes them where
    test_gemm_queues_taken says) and bit-equal to mz_q4_gemm."""
    for i, (M, N, K, epi) in enumerate(_layer_gemms(key)):
        _gemm_case(M, N, K, epi, seed=100 + i, sample_rows=_tile_rows(M, 64, i), n_split="queued")


def _rope_table(max_pos, hd, theta):
    """(cos, sin) of p * theta^(-2i/hd) in fp64, stored as fp32 pairs [max_pos][hd/2]."""
    i = np.arange(hd // 2, dtype=np.float64)
    ang = np.arange(max_pos, dtype=np.float64)[:, None] * theta ** (-2.0 * i / hd)[None, :]
    return np.stack([np.cos(ang), np.sin(ang)], axis=-1).astype(np.float32)


@pytest.mark.parametrize("key", ["1b", "3b", "1p5b", "8b"])
def test_gemm_restore_launches(key):
    """The projections as the restore launches them (mz_q4_gemm_ex), at the
    workload's full row count: with the runtime's 64 MiB workspace, so the
    rows after the last whole 256-row tile run split over K where their tiles
    alone would leave the chip idle; through a row list (a ragged subset of the
    activation rows, as the restore passes R_l / D_l); with the work queues;
    and with the rotary epilogues (queries to f16; keys and values into chunk
    slots).  Against the exact product (and the oracle's rotary embedding) on
    one row in every 64-row tile and both sides of the last whole 256-row
    tile; rows in whole 256-row tiles bit-equal to mz_q4_gemm's."""
    torch = torch_cuda()
    w = W.WORKLOADS[key]
    m = w.model
    S = w.n_ctx + w.n_prompt
    d, hd, C = m.d_model, m.head_dim, m.chunk_tokens
    rng = np.random.default_rng(17)
    gen = torch.Generator(device="cuda").manual_seed(17)
    X = torch.randn(S, d, device="cuda", generator=gen).to(torch.float16)
    Xh = X.float().cpu().numpy().astype(np.float64)
    ws_bytes = 64 << 20
    ws = torch.full((ws_bytes // 4,), float("nan"), device="cuda")
    queues = torch.zeros(16, device="cuda", dtype=torch.int32)
    cs = torch.from_numpy(_rope_table(S, hd, m.rope_theta)).cuda()
    # a ragged row list: every row of a random half of the chunks, then the prompt
    keep = rng.random(w.n_chunks) < 0.5
    sub = np.array([p for p in range(S) if p >= w.n_ctx or keep[p // C]], np.int32)
    d_sub = torch.from_numpy(sub).cuda()
    for rows_name, M, arow, pos_np in (("all", S, None, np.arange(S, dtype=np.int32)), ("list", sub.size, sub, sub)):
        d_pos = torch.from_numpy(np.ascontiguousarray(pos_np)).cuda()
        xr = Xh if arow is None else Xh[arow]
        ar_ptr = 0 if arow is None else d_sub.data_ptr()
        check = _tile_rows(M, 64, M)
        full = M // 256 * 256
        # queries, rotated
        raw = W.encode_q4_0((rng.standard_normal((m.dq, d)) * 0.02).astype(np.float32))
        Wm = O.q4_0_decode(raw.reshape(-1), m.dq, d)
        n_pad = (m.dq + 255) // 256 * 256
        wdev = torch.from_numpy(mz.mz_q4_gemm_pack(raw, m.dq, d)).cuda()
        yq = torch.full((M, m.dq), float("nan"), device="cuda", dtype=torch.float16)
        report("restore launch", workload=key, rows=rows_name, M=M, proj="q-rope")
        mz.mz_q4_gemm_ex(X.data_ptr(), M, n_pad, d, wdev.data_ptr(), 4, yq.data_ptr(), stream(), a_rows=ar_ptr,
                         workspace=ws.data_ptr(), workspace_bytes=ws_bytes, pos=d_pos.data_ptr(),
                         rope_cs=cs.data_ptr(), head_dim=hd, n_valid=m.dq)
        torch.cuda.synchronize()
        xs = xr[check]
        prod = xs @ Wm.T
        b = REL * (np.abs(xs) @ np.abs(Wm).T) + 1e-6
        ref = O.rope(prod.reshape(-1, m.n_q_heads, hd), pos_np[check], m.rope_theta).reshape(-1, m.dq)
        bh = b.reshape(-1, m.n_q_heads, hd)
        bound = (bh + np.concatenate([bh[..., hd // 2:], bh[..., :hd // 2]], -1)).reshape(-1, m.dq)
        bound = bound + F16_REL * np.abs(ref) + 2.0 ** -22 * np.abs(prod).max()
        got = yq.float().cpu().numpy()[check].astype(np.float64)
        err = np.abs(got - ref)
        report("  err", max=float(err.max()), worst_ratio=float((err / bound).max()))
        assert np.all(err <= bound)
        # keys and values into chunk slots
        rk = W.encode_q4_0((rng.standard_normal((m.dkv, d)) * 0.02).astype(np.float32))
        rv = W.encode_q4_0((rng.standard_normal((m.dkv, d)) * 0.02).astype(np.float32))
        Wk, Wv = O.q4_0_decode(rk.reshape(-1), m.dkv, d), O.q4_0_decode(rv.reshape(-1), m.dkv, d)
        n_kv = 2 * m.dkv
        wdev = torch.from_numpy(mz.mz_q4_gemm_pack(np.concatenate([rk, rv]), n_kv, d)).cuda()
        n_slots = (S + C - 1) // C + 1
        slot_bytes = C * m.dkv * 4
        perm = rng.permutation(n_slots)[: (S + C - 1) // C]
        kv_off = (perm[pos_np // C].astype(np.int64) * slot_bytes + (pos_np % C).astype(np.int64) * m.dkv * 2)
        slab = torch.full((n_slots * slot_bytes // 2,), float("nan"), device="cuda", dtype=torch.float16)
        d_off = torch.from_numpy(kv_off).cuda()
        report("restore launch", workload=key, rows=rows_name, M=M, proj="kv-rope-slots")
        mz.mz_q4_gemm_ex(X.data_ptr(), M, (n_kv + 255) // 256 * 256, d, wdev.data_ptr(), 5, 0, stream(),
                         a_rows=ar_ptr, workspace=ws.data_ptr(), workspace_bytes=ws_bytes, pos=d_pos.data_ptr(),
                         rope_cs=cs.data_ptr(), kv_off=d_off.data_ptr(), slab=slab.data_ptr(), head_dim=hd,
                         n_valid=n_kv, chunk_tokens=C)
        torch.cuda.synchronize()
        sl = slab.view(torch.uint8).cpu().numpy()
        pk, pv = xs @ Wk.T, xs @ Wv.T
        bk = REL * (np.abs(xs) @ np.abs(Wk).T) + 1e-6
        bv = REL * (np.abs(xs) @ np.abs(Wv).T) + 1e-6
        kref = O.rope(pk.reshape(-1, m.n_kv_heads, hd), pos_np[check], m.rope_theta).reshape(-1, m.dkv)
        bkh = bk.reshape(-1, m.n_kv_heads, hd)
        kb = (bkh + np.concatenate([bkh[..., hd // 2:], bkh[..., :hd // 2]], -1)).reshape(-1, m.dkv)
        kb = kb + F16_REL * np.abs(kref) + 2.0 ** -22 * np.abs(pk).max()
        vb = bv + F16_REL * np.abs(pv)
        for j, r in enumerate(check):
            off = int(kv_off[r])
            kg = sl[off:off + m.dkv * 2].view(np.float16).astype(np.float64)
            base = off - int(pos_np[r] % C) * m.dkv * 2 + C * m.dkv * 2
            vt = sl[base:base + m.dkv * C * 2].view(np.float16).reshape(m.dkv, C)[:, pos_np[r] % C]
            assert np.all(np.abs(kg - kref[j]) <= kb[j]), (key, rows_name, int(r), "K")
            assert np.all(np.abs(vt.astype(np.float64) - pv[j]) <= vb[j]), (key, rows_name, int(r), "V")
        # plain epilogues (store, residual add, SwiGLU) with queues and workspace,
        # against mz_q4_gemm bit for bit on whole 256-row tiles
        for i, (N, K, epi) in enumerate([(m.d_model, m.dq, 1), (m.d_ffn, m.d_model, 2)]):
            if K != d:
                continue           # the activation rows are [S][d]
            if epi == 2:
                g_ = W.encode_q4_0((rng.standard_normal((N, K)) * 0.02).astype(np.float32))
                u_ = W.encode_q4_0((rng.standard_normal((N, K)) * 0.02).astype(np.float32))
                wdev = torch.from_numpy(mz.mz_q4_gemm_pack(g_, N, K, w_up=u_)).cuda()
                n_pad = 2 * ((N + 127) // 128 * 128)
                y1 = torch.zeros(M, n_pad // 2, device="cuda", dtype=torch.float16)
            else:
                raw = W.encode_q4_0((rng.standard_normal((N, K)) * 0.02).astype(np.float32))
                wdev = torch.from_numpy(mz.mz_q4_gemm_pack(raw, N, K)).cuda()
                n_pad = (N + 255) // 256 * 256
                y1 = torch.randn(M, n_pad, device="cuda", generator=gen)
            y0 = y1.clone()
            xg = X if arow is None else X[d_sub.long()].contiguous()
            report("restore launch", workload=key, rows=rows_name, M=M, proj=f"epi{epi}")
            mz.mz_q4_gemm_ex(X.data_ptr(), M, n_pad, K, wdev.data_ptr(), epi, y1.data_ptr(), stream(), a_rows=ar_ptr,
                             work_queues=queues.data_ptr(), workspace=ws.data_ptr(), workspace_bytes=ws_bytes)
            y2 = y0.clone()
            mz.mz_q4_gemm(xg.data_ptr(), M, n_pad, K, wdev.data_ptr(), epi, y2.data_ptr(), stream())
            torch.cuda.synchronize()
            assert int(queues.abs().sum()) == 0
            assert torch.equal(y1[:full].view(torch.uint8), y2[:full].view(torch.uint8)), (key, rows_name, epi)
            a1 = y1[full:].float().cpu().numpy().astype(np.float64)
            a2 = y2[full:].float().cpu().numpy().astype(np.float64)
            if a1.size:
                scale = np.abs(a2).max() + 1e-3
                assert np.abs(a1 - a2).max() <= 4 * F16_REL * scale, (key, rows_name, epi)


@pytest.mark.parametrize("epi,hd,K", [
    (0, 0, 192), (1, 0, 192), (2, 0, 192), (4, 32, 192), (4, 64, 192), (4, 128, 192), (5, 32, 192), (5, 64, 192),
    (5, 128, 192), (1, 0, 5440), (2, 0, 5440), (4, 128, 5440), (5, 64, 5440)])
def test_gemm_tile_shapes_same_bits(epi, hd, K):
    """A product's first rows by themselves -- so few that they run as 32-, 64-
    or 128-row tiles of 128 columns -- against the same rows of a product
    that fills the chip with 128 x 256 tiles (K 192) or with four whole rounds
    of 256 x 256 tiles (K 5440): bit for bit, with every epilogue, an odd
    number of 64-wide K steps, row counts at the edges of every tile height,
    a row list, and (keys and values) rows that write nothing and positions
    that do not start on a slot."""
    torch = torch_cuda()
    M, N, C = 4096, 16384, 16
    gen = torch.Generator(device="cuda").manual_seed(epi * 10 + hd)
    X = torch.randn(M, K, device="cuda", generator=gen).to(torch.float16)
    W_ = torch.randint(0, 256, (N // 256, K // 64, 9216), device="cuda", dtype=torch.uint8, generator=gen)
    sc = (torch.rand(N // 256, K // 64, 512, device="cuda", generator=gen) * 0.01 + 0.01).to(torch.float16)
    W_[..., 8192:] = sc.view(torch.uint8).view(N // 256, K // 64, 1024)
    rows = torch.randperm(M, device="cuda", generator=gen).to(torch.int32)
    pos = torch.arange(5, 5 + M, device="cuda", dtype=torch.int32)
    slot = C * (N // 2) * 4
    off = (pos.long() // C) * slot + (pos.long() % C) * (N // 2) * 2
    off[3::7] = -1
    cs = torch.randn(M + 5, max(hd // 2, 1), 2, device="cuda", generator=gen)
    y0 = torch.randn(M, N, device="cuda", generator=gen) if epi < 2 else None

    def run(m):
        slab = torch.zeros((M + 5 + C) // C * slot // 2, device="cuda", dtype=torch.float16) if epi == 5 else None
        y = y0[:m].clone() if epi < 2 else torch.zeros(m, N // 2 if epi == 2 else N, device="cuda", dtype=torch.float16)
        mz.mz_q4_gemm_ex(X.data_ptr(), m, N, K, W_.data_ptr(), epi, 0 if epi == 5 else y.data_ptr(), stream(),
                         a_rows=rows.data_ptr(), pos=pos.data_ptr(), rope_cs=cs.data_ptr(),
                         kv_off=off.data_ptr(), slab=slab.data_ptr() if epi == 5 else 0, head_dim=hd, n_valid=N,
                         chunk_tokens=C)
        torch.cuda.synchronize()
        return slab.view(-1, 2, slot // 4) if epi == 5 else y

    assert mz.mz_q4_gemm_plan(M, N, K) == [(M, 128 if K == 192 else 256, 256, 1)]
    small = {mz.mz_q4_gemm_plan(m, N, K)[0][1:3] for m in (1, 65, 129)}
    assert small == {(32, 128), (64, 128), (128, 128)}
    full = run(M)
    assert bool((full != 0).any())
    for m in (1, 2, 31, 32, 33, 64, 65, 127, 128, 129, 300):
        got = run(m)
        if epi != 5:
            assert torch.equal(got.view(torch.uint8), full[:m].view(torch.uint8)), m
            continue
        p = pos[:m].long()
        written = off[:m] >= 0
        for half, view in ((0, lambda t: t[:, 0].view(-1, C, N // 2)),
                           (1, lambda t: t[:, 1].view(-1, N // 2, C).transpose(1, 2))):
            a, b = view(got), view(full)
            assert torch.equal(a[p // C, p % C][written], b[p // C, p % C][written]), (m, half)
            mask = torch.zeros(a.shape[:2], dtype=torch.bool, device="cuda")
            mask[(p // C)[written], (p % C)[written]] = True
            assert not bool((a[~mask] != 0).any()), (m, half)      # nothing else was written


def _byte_view(t, shift):
    """A copy of t that starts `shift` bytes after a 256-byte boundary, and
    the buffer around it (0x55 bytes elsewhere)."""
    torch = torch_cuda()
    raw = t.reshape(-1).view(torch.uint8)
    buf = torch.full((raw.numel() + 512,), 0x55, device="cuda", dtype=torch.uint8)
    buf[256 + shift:256 + shift + raw.numel()] = raw
    return buf, buf.data_ptr() + 256 + shift


@pytest.mark.parametrize("m", [17, 200])
@pytest.mark.parametrize("epi,hd", [(0, 0), (1, 0), (2, 0), (4, 64), (5, 128)])
def test_gemm_unaligned_operands(m, epi, hd):
    """Outputs that start at any element take the same tiles and K splits as
    aligned ones: the same bits, nothing written beside them.  Weights off a
    16-byte boundary run as 256-row tiles: without a workspace the same bits,
    with one the K splits may be others (fp32 sums in another order)."""
    torch = torch_cuda()
    K, N, C = 2048, 1024, 16
    gen = torch.Generator(device="cuda").manual_seed(epi)
    X = torch.randn(m, K, device="cuda", generator=gen).half()
    W_ = torch.randint(0, 256, (N // 256, K // 64, 9216), device="cuda", dtype=torch.uint8, generator=gen)
    sc = (torch.rand(N // 256, K // 64, 512, device="cuda", generator=gen) * 0.01 + 0.01).half()
    W_[..., 8192:] = sc.view(torch.uint8).view(N // 256, K // 64, 1024)
    pos = torch.arange(5, 5 + m, device="cuda", dtype=torch.int32)
    slot = C * (N // 2) * 4
    off = (pos.long() // C) * slot + (pos.long() % C) * N
    cs = torch.randn(m + 5, max(hd // 2, 1), 2, device="cuda", generator=gen)
    if epi < 2:
        y0 = torch.randn(m, N, device="cuda", generator=gen)
    elif epi == 5:
        y0 = torch.zeros((m + 5 + C) // C * slot // 2, device="cuda", dtype=torch.float16)
    else:
        y0 = torch.zeros(m, N // 2 if epi == 2 else N, device="cuda", dtype=torch.float16)
    wsb = 64 << 20

    def run(y_shift, w_shift, split):
        buf, yp = _byte_view(y0, y_shift)
        wbuf, wp = _byte_view(W_, w_shift)
        ws = torch.full((wsb // 4,), float("nan"), device="cuda")
        kw = dict(workspace=ws.data_ptr(), workspace_bytes=wsb) if split else {}
        report("unaligned", epi=epi, m=m, y_shift=y_shift, w_shift=w_shift, split=split)
        mz.mz_q4_gemm_ex(X.data_ptr(), m, N, K, wp, epi, 0 if epi == 5 else yp, stream(), pos=pos.data_ptr(),
                         rope_cs=cs.data_ptr(), kv_off=off.data_ptr(), slab=yp if epi == 5 else 0, head_dim=hd,
                         n_valid=N, chunk_tokens=C, **kw)
        torch.cuda.synchronize()
        n = y0.numel() * y0.element_size()
        assert bool((buf[:256 + y_shift] == 0x55).all()) and bool((buf[256 + y_shift + n:] == 0x55).all())
        return buf[256 + y_shift:256 + y_shift + n].clone()

    esz = y0.element_size()
    for split in (False, True):
        ref = run(0, 0, split)
        for shift in (esz, 8 + esz):
            assert torch.equal(run(shift, 0, split), ref), (split, shift)
        for shift in (2, 8):
            got = run(0, shift, split)
            if not split:
                assert torch.equal(got, ref), shift
                continue
            a, b = got.view(y0.dtype).double(), ref.view(y0.dtype).double()
            # the order of K fp32 sums, and for halves one rounding that may fall the other way
            tol = K * 2.0 ** -24 if esz == 4 else 2.0 ** -10
            assert float((a - b).abs().max()) <= tol * float(b.abs().max()), shift


def _single_row_shapes(key):
    m = W.WORKLOADS[key].model
    ffp = (m.d_ffn + 127) // 128 * 128      # the SwiGLU output width, as the down projection reads it
    return [("q-rope", m.dq, m.d_model, 4), ("kv-rope-slots", 2 * m.dkv, m.d_model, 5),
            ("q-store", m.dq, m.d_model, 0), ("o-add", m.d_model, m.dq, 1),
            ("gateup-swiglu", m.d_ffn, m.d_model, 2), ("down-add", m.d_model, ffp, 1)]


@pytest.mark.parametrize("key", ["tiny", "1b", "3b", "1p5b", "8b"])
def test_gemv_single_row(key):
    """mz_q4_gemv, the one-launch single-row product (decode steps), for every
    projection of the workload at its full shape, with each epilogue the
    runtime gives it: against the exact product of the decoded weights (and
    the oracle's rotary embedding) on every output column, for a row picked
    from a matrix through a_rows; the RMSNorm-forming variant against the
    same product of mz_rmsnorm's output, bit for bit."""
    torch = torch_cuda()
    w = W.WORKLOADS[key]
    m = w.model
    hd, C = m.head_dim, m.chunk_tokens
    rng = np.random.default_rng(23)
    gen = torch.Generator(device="cuda").manual_seed(23)
    n_rows = 5
    row = 3
    d_row = torch.tensor([row], device="cuda", dtype=torch.int32)
    p = int(w.n_ctx + w.n_prompt - 1)                 # the position of a decode row
    cs = torch.from_numpy(_rope_table(p + 1, hd, m.rope_theta)).cuda()
    d_pos = torch.tensor([p], device="cuda", dtype=torch.int32)
    for name, N, K, epi in _single_row_shapes(key):
        report("gemv", workload=key, proj=name, N=N, K=K, epi=epi)
        X = torch.randn(n_rows, K, device="cuda", generator=gen).to(torch.float16)
        xs = X[row].float().cpu().numpy().astype(np.float64)[None, :]
        if epi == 2:
            g_ = W.encode_q4_0((rng.standard_normal((N, K)) * 0.02).astype(np.float32))
            u_ = W.encode_q4_0((rng.standard_normal((N, K)) * 0.02).astype(np.float32))
            wdev = torch.from_numpy(mz.mz_q4_gemm_pack(g_, N, K, w_up=u_)).cuda()
            n_pad = 2 * ((N + 127) // 128 * 128)
            G, U = O.q4_0_decode(g_.reshape(-1), N, K), O.q4_0_decode(u_.reshape(-1), N, K)
        elif epi == 5:
            half_n = N // 2
            rk = W.encode_q4_0((rng.standard_normal((half_n, K)) * 0.02).astype(np.float32))
            rv = W.encode_q4_0((rng.standard_normal((half_n, K)) * 0.02).astype(np.float32))
            wdev = torch.from_numpy(mz.mz_q4_gemm_pack(np.concatenate([rk, rv]), N, K)).cuda()
            n_pad = (N + 255) // 256 * 256
            Wk, Wv = O.q4_0_decode(rk.reshape(-1), half_n, K), O.q4_0_decode(rv.reshape(-1), half_n, K)
        else:
            raw = W.encode_q4_0((rng.standard_normal((N, K)) * 0.02).astype(np.float32))
            wdev = torch.from_numpy(mz.mz_q4_gemm_pack(raw, N, K)).cuda()
            n_pad = (N + 255) // 256 * 256
            Wm = O.q4_0_decode(raw.reshape(-1), N, K)

        def run(x_ptr, h_ptr, out):
            kw = dict(a_rows=d_row.data_ptr(), h_norm=h_ptr, eps=float(m.rms_eps))
            if epi == 4:
                kw.update(pos=d_pos.data_ptr(), rope_cs=cs.data_ptr(), head_dim=hd, n_valid=N)
            if epi == 5:
                kw.update(pos=d_pos.data_ptr(), rope_cs=cs.data_ptr(), kv_off=d_off.data_ptr(),
                          slab=out.data_ptr(), head_dim=hd, n_valid=N, chunk_tokens=C)
            mz.mz_q4_gemv(x_ptr, K, wdev.data_ptr(), n_pad, epi, 0 if epi == 5 else out.data_ptr(), stream(),
                          **kw)

        if epi == 5:
            slot_bytes = C * (N // 2) * 4
            slot, pc = 2, p % C
            out = torch.full((4 * slot_bytes // 2,), float("nan"), device="cuda", dtype=torch.float16)
            d_off = torch.tensor([slot * slot_bytes + pc * (N // 2) * 2], device="cuda", dtype=torch.int64)
        elif epi == 4:
            out = torch.full((1, N), float("nan"), device="cuda", dtype=torch.float16)
        elif epi == 2:
            out = torch.full((1, n_pad // 2), float("nan"), device="cuda", dtype=torch.float16)
        elif epi == 1:
            out = torch.randn(1, n_pad, device="cuda", generator=gen)
        else:
            out = torch.full((1, n_pad), float("nan"), device="cuda")
        out0 = out.clone()
        run(X.data_ptr(), 0, out)
        torch.cuda.synchronize()
        if epi == 4:
            prod = xs @ Wm.T
            b = REL * (np.abs(xs) @ np.abs(Wm).T) + 1e-6
            ref = O.rope(prod.reshape(1, m.n_q_heads, hd), np.array([p]), m.rope_theta).reshape(1, N)
            bh = b.reshape(1, m.n_q_heads, hd)
            bound = (bh + np.concatenate([bh[..., hd // 2:], bh[..., :hd // 2]], -1)).reshape(1, N)
            bound = bound + F16_REL * np.abs(ref) + 2.0 ** -22 * np.abs(prod).max()
            got = out.float().cpu().numpy().astype(np.float64)
        elif epi == 5:
            dkv = N // 2
            pk, pv = xs @ Wk.T, xs @ Wv.T
            bk = REL * (np.abs(xs) @ np.abs(Wk).T) + 1e-6
            bv = REL * (np.abs(xs) @ np.abs(Wv).T) + 1e-6
            kref = O.rope(pk.reshape(1, m.n_kv_heads, hd), np.array([p]), m.rope_theta).reshape(1, dkv)
            bkh = bk.reshape(1, m.n_kv_heads, hd)
            kb = (bkh + np.concatenate([bkh[..., hd // 2:], bkh[..., :hd // 2]], -1)).reshape(1, dkv)
            kb = kb + F16_REL * np.abs(kref) + 2.0 ** -22 * np.abs(pk).max()
            sl = out.view(torch.uint8).cpu().numpy()
            off = slot * slot_bytes + pc * dkv * 2
            kg = sl[off:off + dkv * 2].view(np.float16).astype(np.float64)[None, :]
            base = slot * slot_bytes + C * dkv * 2
            vt = sl[base:base + dkv * C * 2].view(np.float16).reshape(dkv, C)[:, pc].astype(np.float64)[None, :]
            got = np.concatenate([kg, vt], 1)
            ref = np.concatenate([kref, pv], 1)
            bound = np.concatenate([kb, bv + F16_REL * np.abs(pv)], 1)
            # nothing else of the slab was written
            touched = np.zeros(sl.size // 2, bool)
            touched[off // 2: off // 2 + dkv] = True
            touched[base // 2 + np.arange(dkv) * C + pc] = True
            assert np.all(np.isnan(out.float().cpu().numpy()[~touched]))
        elif epi == 2:
            gr, ur = xs @ G.T, xs @ U.T
            bg = REL * (np.abs(xs) @ np.abs(G).T) + 1e-6
            bu = REL * (np.abs(xs) @ np.abs(U).T) + 1e-6
            ref = O.silu(gr) * ur
            bound = 1.1 * bg * (np.abs(ur) + bu) + np.abs(O.silu(gr)) * bu + REL * np.abs(ref) + 1e-6
            ys = out.float().cpu().numpy().astype(np.float64)
            got = ys[:, :N]
            assert np.all(ys[:, N:] == 0)          # padded gate/up columns give silu(0) * 0
        else:
            ref = xs @ Wm.T + (out0.cpu().numpy().astype(np.float64)[:, :N] if epi == 1 else 0.0)
            bound = REL * (np.abs(xs) @ np.abs(Wm).T) + 1e-5 * (1 + np.abs(ref))
            got = out.cpu().numpy().astype(np.float64)[:, :N]
        err = np.abs(got - ref)
        report("  err", max=float(err.max()), worst_ratio=float((err / bound).max()))
        assert np.all(err <= bound), (key, name)
        # the RMSNorm-forming variant: the same bits as the product of mz_rmsnorm's rows
        if K == m.d_model:
            H = torch.randn(n_rows, K, device="cuda", generator=gen) * 3.0
            Xn = torch.empty(n_rows, K, device="cuda", dtype=torch.float16)
            mz.mz_rmsnorm(H.data_ptr(), n_rows, K, float(m.rms_eps), Xn.data_ptr(), stream())
            o1, o2 = out0.clone(), out0.clone()
            if epi == 5:
                o1.fill_(float("nan"))
                o2.fill_(float("nan"))
            run(Xn.data_ptr(), 0, o1)
            run(0, H.data_ptr(), o2)
            torch.cuda.synchronize()
            assert torch.equal(o1.view(torch.uint8), o2.view(torch.uint8)), (key, name, "norm in gemv")


def test_gemv_validation():
    torch = torch_cuda()
    x = torch.zeros(1, 256, device="cuda", dtype=torch.float16)
    w = torch.zeros(mz.mz_q4_gemm_packed_bytes(256, 256), device="cuda", dtype=torch.uint8)
    y = torch.zeros(1, 256, device="cuda")
    bad = [dict(k=256, n_pad=100, epi=0), dict(k=100, n_pad=256, epi=0), dict(k=16448, n_pad=256, epi=0),
           dict(k=256, n_pad=256, epi=3), dict(k=256, n_pad=256, epi=4)]
    for b in bad:
        with pytest.raises(mz.MzError):
            mz.mz_q4_gemv(x.data_ptr(), b["k"], w.data_ptr(), b["n_pad"], b["epi"], y.data_ptr(), stream())
    with pytest.raises(mz.MzError):
        mz.mz_q4_gemv(x.data_ptr(), 256, w.data_ptr(), 256, 0, y.data_ptr(), stream(), h_norm=y.data_ptr(),
                      eps=-1.0)


@pytest.mark.parametrize("M,N,K,epi", [
    (20000, 14336, 128, 0), (16640, 16384, 64, 1), (20000, 7168, 128, 2), (33000, 8192, 64, 1),
    (1000, 2048, 512, 0), (9000, 4096, 512, 1), (300, 512, 128, 1)])
def test_gemm_queued(M, N, K, epi):
    """mz_q4_gemm_queued for every plain epilogue on products that run in
    other tiles than 256 x 256, short K ranges of many rounds and small ones:
    the queues stay untouched, one workgroup per tile (test_gemm_queues_taken
    has the products that take them).  Against the exact product on sampled
    rows and bit-equal to mz_q4_gemm."""
    assert all(p[1:3] != (256, 256) for p in mz.mz_q4_gemm_plan(M, 2 * N if epi == 2 else N, K, 0, True))
    rows = None
    if M > 4000:
        rng = np.random.default_rng(M)
        rows = np.unique(np.concatenate([rng.choice(M, 40, replace=False),
                                         [0, M // 256 * 256 - 1, M // 256 * 256, M - 1]]))
        rows = rows[rows < M]   # M // 256 * 256 is M itself when M is a multiple of 256
    _gemm_case(M, N, K, epi, seed=M + 7, sample_rows=rows, n_split="queued")


@pytest.mark.parametrize("M,epi", [(16400, 0), (16384, 1), (16400, 2)])
def test_gemm_queues_taken(M, epi):
    """Products whose plan is 256 x 256 tiles, 16 rounds of them and more (4096
    tiles), take the work queues in the store, residual-add and SwiGLU
    epilogue, with and without a ragged remainder in a second launch: the
    bits of mz_q4_gemm, which runs them one workgroup per tile, and of the
    rows at tile edges by themselves (32-row tiles); the queues come back
    zero, twice."""
    torch = torch_cuda()
    N, K = 16384, 6016
    plan = mz.mz_q4_gemm_plan(M, N, K, 0, True)
    assert plan[0] == (16384, 256, 256, 1) and 16384 // 256 * (N // 256) >= 4096, plan
    gen = torch.Generator(device="cuda").manual_seed(M + epi)
    X = torch.randn(M, K, device="cuda", generator=gen).half()
    W_ = torch.randint(0, 256, (N // 256, K // 64, 9216), device="cuda", dtype=torch.uint8, generator=gen)
    sc = (torch.rand(N // 256, K // 64, 512, device="cuda", generator=gen) * 0.01 + 0.01).half()
    W_[..., 8192:] = sc.view(torch.uint8).view(N // 256, K // 64, 1024)
    if epi == 1:
        y0 = torch.randn(M, N, device="cuda", generator=gen)
    else:
        y0 = torch.zeros(M, N // 2 if epi == 2 else N, device="cuda", dtype=torch.float16 if epi == 2 else torch.float32)
    plain = y0.clone()
    report("queues taken", M=M, epi=epi, plan=plan)
    mz.mz_q4_gemm(X.data_ptr(), M, N, K, W_.data_ptr(), epi, plain.data_ptr(), stream())
    queues = torch.zeros(16, device="cuda", dtype=torch.int32)
    y = torch.empty_like(y0)
    for _ in range(2):
        y.copy_(y0)
        mz.mz_q4_gemm_queued(X.data_ptr(), M, N, K, W_.data_ptr(), epi, y.data_ptr(), queues.data_ptr(), stream())
        torch.cuda.synchronize()
        assert int(queues.abs().sum()) == 0, "work queues not left at zero"
        assert torch.equal(y, plain), "queued != mz_q4_gemm"
    rows = torch.tensor([0, 255, 256, 5000, 8191, 8192, 16383, M - 1], device="cuda")
    few = y0[rows].contiguous()
    mz.mz_q4_gemm(X[rows].contiguous().data_ptr(), len(rows), N, K, W_.data_ptr(), epi, few.data_ptr(), stream())
    torch.cuda.synchronize()
    assert bool((few != 0).any()) and torch.equal(few, y[rows])


def _attn_case(nq, nkv, hd, C, S, qpos, seed, sample=None, n_split=None, n_table=None):
    """n_split: None for mz_attention, "queued" for mz_attention_queued (run
    twice on the same queues, which must come back zero, and equal to
    mz_attention bit for bit), else mz_attention_split with that many key
    splits ("auto": the restore's choice)."""
    torch = torch_cuda()
    report("attention", nq=nq, nkv=nkv, hd=hd, C=C, S=S, m=len(qpos), seed=seed, n_split=n_split)
    if sample is not None:
        assert 0 <= int(np.min(sample)) and int(np.max(sample)) < len(qpos), "sample rows out of range"
    rng = np.random.default_rng(seed)
    dkv = nkv * hd
    nch = (S + C - 1) // C
    n_slots = nch + 3
    table = rng.permutation(n_slots)[:nch].astype(np.int32)
    K = rng.standard_normal((S, dkv)).astype(np.float16)
    V = rng.standard_normal((S, dkv)).astype(np.float16)
    # slot: K [C][dkv] token-major, then V^T [dkv][C]; unused rows are NaN
    kpart = np.full((n_slots, C, dkv), np.nan, np.float16)
    vpart = np.full((n_slots, dkv, C), np.nan, np.float16)
    for c in range(nch):
        n = min(C, S - c * C)
        kpart[table[c], :n] = K[c * C:c * C + n]
        vpart[table[c], :, :n] = V[c * C:c * C + n].T
    slab = np.concatenate([kpart.reshape(n_slots, -1), vpart.reshape(n_slots, -1)], axis=1)
    if n_table is not None:
        # a longer table than the keys need (entries past them name slot 0)
        table = np.concatenate([table, np.zeros(n_table - nch, np.int32)])
        nch = n_table
    qpos = np.asarray(qpos, np.int32)
    M = qpos.size
    q = (rng.standard_normal((M, nq, hd)) * 1.0).astype(np.float16)
    d_q = torch.from_numpy(q).cuda()
    d_pos = torch.from_numpy(qpos).cuda()
    d_slab = torch.from_numpy(slab).cuda()
    d_tab = torch.from_numpy(table).cuda()
    out = torch.empty(M, nq * hd, device="cuda", dtype=torch.float16)
    max_pos = int(qpos[-1])
    if n_split is None:
        mz.mz_attention(d_q.data_ptr(), d_pos.data_ptr(), M, d_slab.data_ptr(), d_tab.data_ptr(), nch, C,
                        nq, nkv, hd, out.data_ptr(), stream())
    elif n_split == "queued":
        queues = torch.zeros(16, device="cuda", dtype=torch.int32)
        plain = torch.empty_like(out)
        mz.mz_attention(d_q.data_ptr(), d_pos.data_ptr(), M, d_slab.data_ptr(), d_tab.data_ptr(), nch, C,
                        nq, nkv, hd, plain.data_ptr(), stream())
        for rep in range(2):
            out.fill_(float("nan"))
            mz.mz_attention_queued(d_q.data_ptr(), d_pos.data_ptr(), M, d_slab.data_ptr(), d_tab.data_ptr(), nch,
                                   C, nq, nkv, hd, out.data_ptr(), queues.data_ptr(), stream())
            torch.cuda.synchronize()
            assert int(queues.abs().sum()) == 0, "work queues not left at zero"
            assert torch.equal(out.view(torch.int16), plain.view(torch.int16)), "queued != mz_attention"
    else:
        if n_split == "auto":
            n_split = mz.mz_attention_auto_splits(M, max_pos, nq, nkv, hd, 64 << 20)
            report("  auto splits", n_split=n_split)
        wsb = mz.mz_attention_split_workspace_bytes(M, nq, hd, n_split)
        ws = torch.empty(wsb, device="cuda", dtype=torch.uint8)
        mz.mz_attention_split(d_q.data_ptr(), d_pos.data_ptr(), M, max_pos, d_slab.data_ptr(), d_tab.data_ptr(),
                              nch, C, nq, nkv, hd, n_split, ws.data_ptr(), wsb, out.data_ptr(), stream())
    torch.cuda.synchronize()
    got = out.float().cpu().numpy().reshape(M, nq, hd).astype(np.float64)
    rows = np.arange(M) if sample is None else sample
    ref = O.causal_gqa_attention(q[rows].astype(np.float64), qpos[rows],
                                 K.astype(np.float64).reshape(S, nkv, hd),
                                 V.astype(np.float64).reshape(S, nkv, hd))
    g = got[rows]
    bound = REL * np.abs(ref) + 2.0 ** -10 * float(np.abs(V).max())
    if n_split is not None:
        # each split's normalised output is a convex combination of V rows,
        # rounded to f16 (half an ulp: 2^-11 max|V|); the merge is again a
        # convex combination of those
        bound = bound + 2.0 ** -11 * float(np.abs(V).max())
    err = np.abs(g - ref)
    report("  err", max=float(err.max()), worst_ratio=float((err / bound).max()))
    assert np.all(np.isfinite(g))
    assert np.all(err <= bound)


@pytest.mark.parametrize("nq,nkv,hd,C,S", [
    (4, 2, 64, 16, 128), (4, 2, 64, 16, 117), (32, 8, 64, 256, 600), (24, 8, 128, 256, 700),
    (12, 2, 128, 256, 530), (32, 8, 128, 256, 400), (8, 8, 128, 64, 200), (6, 1, 64, 32, 90),
    (4, 4, 128, 8, 77), (10, 2, 64, 64, 450), (14, 2, 128, 128, 600), (16, 2, 64, 32, 333)])
def test_attention_small(nq, nkv, hd, C, S):
    """Query-head groups of 1-8 (so every wave map: G heads x 8/G row groups,
    2 heads x 4 for G = 6, one head x 8 for G = 3, 5, 7), dense, gappy, first
    and last query rows, against the exact definition."""
    rng = np.random.default_rng(S)
    dense = np.arange(S)
    gappy = np.sort(rng.choice(S, max(1, S // 3), replace=False))
    _attn_case(nq, nkv, hd, C, S, dense, seed=1)
    _attn_case(nq, nkv, hd, C, S, gappy, seed=2)
    _attn_case(nq, nkv, hd, C, S, [0], seed=3)
    _attn_case(nq, nkv, hd, C, S, [S - 1], seed=4)


@pytest.mark.parametrize("key", ["1b", "3b", "1p5b", "8b"])
def test_attention_full_context(key):
    """All S query rows of the workload through the work queues (the
    restore's launch), bit-equal to the one-tile-per-workgroup form, and one
    query row (every head, so every KV head) in every 32-row query tile
    checked against the exact definition."""
    w = W.WORKLOADS[key]
    m = w.model
    S = w.n_ctx + w.n_prompt
    _attn_case(m.n_q_heads, m.n_kv_heads, m.head_dim, m.chunk_tokens, S, np.arange(S), seed=5,
               sample=_tile_rows(S, 32, 5), n_split="queued")


def test_attention_full_context_gappy_1p5b():
    """The 1.5B shape (12 query / 2 KV heads, head dim 128) at its full
    16384-token context with gappy query rows: the rows of a seeded 30 % of
    the chunks (a recompute's R_l), through the work queues; one query in
    every 32-row tile checked."""
    w = W.WORKLOADS["1p5b"]
    m = w.model
    S = w.n_ctx
    rng = np.random.default_rng(31)
    keep = rng.random(w.n_chunks) < 0.3
    qpos = np.array([p for p in range(S) if keep[p // m.chunk_tokens] or p == S - 1], np.int32)
    _attn_case(m.n_q_heads, m.n_kv_heads, m.head_dim, m.chunk_tokens, S, qpos, seed=6,
               sample=_tile_rows(qpos.size, 32, 6), n_split="queued")


@pytest.mark.parametrize("nq,nkv,hd,C,S", [
    (32, 8, 128, 256, 3000), (24, 8, 128, 256, 1700), (12, 2, 128, 256, 1030), (16, 4, 64, 64, 900),
    (8, 8, 128, 64, 200), (6, 1, 64, 128, 700), (12, 3, 64, 256, 600), (4, 4, 128, 8, 77)])
def test_attention_queued(nq, nkv, hd, C, S):
    """mz_attention_queued with 1, 2, 4 and 8 KV heads, gappy query rows and a
    single one, up to one and a half rounds of workgroups: those take the
    one-tile-per-workgroup form, as 3 KV heads and 8-token chunks always do
    (test_attention_queues_taken has the launches that take the queues)."""
    rng = np.random.default_rng(S + 1)
    gappy = np.sort(rng.choice(S, max(1, S // 3), replace=False))
    _attn_case(nq, nkv, hd, C, S, np.arange(S), seed=11, n_split="queued")
    _attn_case(nq, nkv, hd, C, S, gappy, seed=12, n_split="queued")
    _attn_case(nq, nkv, hd, C, S, [S - 1], seed=13, n_split="queued")


@pytest.mark.parametrize("nq,nkv,hd,C,m", [(32, 8, 128, 64, 3073), (16, 4, 64, 128, 6200), (12, 2, 128, 256, 8200),
                                           (7, 1, 64, 64, 14100), (8, 1, 128, 256, 700), (16, 2, 64, 64, 12000)])
def test_attention_queues_taken(nq, nkv, hd, C, m):
    """Launches that take the work queues: more than 98304 (row, head) pairs
    with 1, 2, 4 and 8 KV heads (queues shared by 8, 4, 2 and 1 XCDs), and
    groups of 8 heads, which take them at any size (fewer tiles than
    workgroups among them).  Rows spread over twice as many positions, once
    with the longest chunk table; the bits of mz_attention, queues left zero,
    sampled rows exact."""
    assert m * nq > 98304 or nq // nkv == 8
    rng = np.random.default_rng(m)
    qpos = np.sort(rng.choice(2 * m, m, replace=False)).astype(np.int32)
    _attn_case(nq, nkv, hd, C, 2 * m, qpos, seed=m, sample=rng.choice(m, 24, replace=False), n_split="queued",
               n_table=8192 if m == 3073 else None)


def test_attention_max_table():
    """A chunk table of 8192 entries, the most the attention entry points
    take (its stretch for each work item is copied into LDS): the plain, the
    work-queue and the split forms against the exact definition."""
    for n_split in (None, "queued", 4):
        _attn_case(32, 8, 128, 64, 700, np.arange(700), seed=41, n_split=n_split, n_table=8192)


@pytest.mark.parametrize("nq,nkv,hd,C,S", [
    (4, 2, 64, 16, 700), (32, 8, 128, 256, 2000), (24, 8, 128, 256, 1500), (12, 2, 128, 256, 1100),
    (8, 8, 128, 64, 900), (6, 1, 64, 32, 800), (4, 4, 128, 8, 333)])
def test_attention_split(nq, nkv, hd, C, S):
    """Split-key attention against the exact definition: prompt-like tails,
    one row, rows far apart (early rows see no key of the later splits), and
    a row at position 0; 2..64 splits (one tile per split at the top)."""
    rng = np.random.default_rng(S + nq)
    cases = [np.arange(S - 9, S), [S - 1], [3, S // 2, S - 1], np.concatenate([[10], np.arange(S - 70, S)]),
             np.sort(rng.choice(S, 40, replace=False)), [0]]
    for i, qp in enumerate(cases):
        for n_split in (2, 5, "auto", 64):
            _attn_case(nq, nkv, hd, C, S, qp, seed=20 + i, n_split=n_split)


@pytest.mark.parametrize("nq,nkv,hd,C,S,m", [(6, 2, 128, 64, 1500, 343), (8, 2, 64, 64, 4200, 300),
                                            (4, 4, 64, 16, 900, 513)])
def test_attention_split_many_pairs(nq, nkv, hd, C, S, m):
    """From 2048 (row, head) pairs on the merge takes 16 (head dimension 128)
    or 32 pairs per workgroup: a ragged last workgroup, rows that see one
    split next to rows that see all of them, and split counts at the edges of
    a pair's lanes (8 and 16) and of its batches of 4."""
    rng = np.random.default_rng(S)
    rows = np.sort(rng.choice(S - 1, m - 2, replace=False) + 1)
    qp = np.concatenate([[0], rows, [S - 1]])
    sample = np.unique(np.concatenate([[0, 1, m - 2, m - 1], rng.integers(0, m, 60)]))
    for n_split in (2, 7, 9, 14, 60):
        _attn_case(nq, nkv, hd, C, S, qp, seed=n_split, sample=sample, n_split=n_split)


@pytest.mark.parametrize("m", [100, 400])
def test_attention_split_nonfinite_values(m):
    """An infinite and a NaN value under keys whose weight underflows to 0 (the
    score lies 369 powers of two below the others): the value's dimension is
    not finite in the plain form, where 0 * inf is NaN, and so it has to be in
    either merge (400 rows of 8 heads: many pairs per workgroup; 100: one
    each); every other dimension is the plain form's to the f16 rounding of
    the partials."""
    torch = torch_cuda()
    nq, nkv, hd, C, S, n_split = 8, 2, 64, 64, 1024, 8
    n = S // C
    gen = torch.Generator(device="cuda").manual_seed(m)
    K = torch.full((n, C, nkv * hd), 4.0, device="cuda")
    K[:2] = -4.0                                         # the first split: keys 0..127
    V = torch.randn(n, nkv * hd, C, device="cuda", generator=gen)
    V[0, 3, 5], V[1, 17, 9] = float("inf"), float("nan")   # both of KV head 0
    slab = torch.cat([K.reshape(n, -1), V.reshape(n, -1)], 1).half()
    table = torch.arange(n, device="cuda", dtype=torch.int32)
    q = torch.full((m, nq * hd), 4.0, device="cuda", dtype=torch.float16)
    pos = torch.arange(S - m, S, device="cuda", dtype=torch.int32)
    args = (slab.data_ptr(), table.data_ptr(), n, C, nq, nkv, hd)
    plain, split = torch.zeros_like(q), torch.zeros_like(q)
    mz.mz_attention(q.data_ptr(), pos.data_ptr(), m, *args, plain.data_ptr(), stream())
    wsb = mz.mz_attention_split_workspace_bytes(m, nq, hd, n_split)
    ws = torch.empty(wsb, device="cuda", dtype=torch.uint8)
    mz.mz_attention_split(q.data_ptr(), pos.data_ptr(), m, S - 1, *args, n_split, ws.data_ptr(), wsb,
                          split.data_ptr(), stream())
    torch.cuda.synchronize()
    bad = torch.zeros(m, nq, hd, dtype=torch.bool, device="cuda")
    bad[:, :nq // nkv, [3, 17]] = True
    assert torch.equal(~torch.isfinite(plain.view(m, nq, hd)), bad)
    assert torch.equal(~torch.isfinite(split.view(m, nq, hd)), bad)
    ok = ~bad.view(m, -1)
    vmax = float(V[torch.isfinite(V)].abs().max())       # partials and results are convex combinations of values
    # each form lies within 2^-10 vmax of the exact rows, the split one 2^-11 more for its partials, and outputs round to f16
    assert float((split - plain)[ok].abs().max()) <= 3 * 2.0 ** -10 * vmax


@pytest.mark.parametrize("m", [2, 100, 400])
def test_attention_split_nan_keys(m):
    """A NaN key makes every output of its KV head NaN in the plain form, and
    so in the split form (2 rows: the few-column kernel; 100 and 400: the tiled
    one with either merge): a range whose sum is NaN is not one without keys.
    Two NaN keys, one among other keys of its range and one range whose keys
    are all NaN; the other KV head is untouched."""
    torch = torch_cuda()
    nq, nkv, hd, C, S, n_split = 8, 2, 64, 64, 1024, 8
    n = S // C
    gen = torch.Generator(device="cuda").manual_seed(m)
    q = torch.randn(m, nq * hd, device="cuda", generator=gen).half()
    table = torch.arange(n, device="cuda", dtype=torch.int32)
    pos = torch.arange(S - m, S, device="cuda", dtype=torch.int32)
    wsb = mz.mz_attention_split_workspace_bytes(m, nq, hd, n_split)
    for whole in (False, True):
        K = torch.randn(n, C, nkv * hd, device="cuda", generator=gen)
        V = torch.randn(n, nkv * hd, C, device="cuda", generator=gen)
        if whole:
            K[2:4, :, :hd] = float("nan")                # keys 128..255: one range of eight
        else:
            K[1, 7, 3] = float("nan")
        slab = torch.cat([K.reshape(n, -1), V.reshape(n, -1)], 1).half()
        args = (slab.data_ptr(), table.data_ptr(), n, C, nq, nkv, hd)
        plain, split = torch.zeros_like(q), torch.zeros_like(q)
        mz.mz_attention(q.data_ptr(), pos.data_ptr(), m, *args, plain.data_ptr(), stream())
        ws = torch.empty(wsb, device="cuda", dtype=torch.uint8)
        mz.mz_attention_split(q.data_ptr(), pos.data_ptr(), m, S - 1, *args, n_split, ws.data_ptr(), wsb,
                              split.data_ptr(), stream())
        torch.cuda.synchronize()
        half = nq // nkv * hd
        for o in (plain, split):
            assert bool(torch.isnan(o[:, :half]).all()) and bool(torch.isfinite(o[:, half:]).all()), whole


@pytest.mark.parametrize("nq,nkv,hd,C,line", [(32, 8, 128, 64, 3072), (24, 8, 128, 256, 4096), (48, 8, 64, 64, 2048),
                                              (32, 8, 64, 16, 1024), (40, 8, 128, 128, 2457)])
def test_attention_wave_count_line(nq, nkv, hd, C, line):
    """Up to `line` rows an unsplit launch takes workgroups of four waves,
    above it of eight (groups 4, 3, 6, 4 and 5): first and last rows, tile
    edges of both and a ragged last tile, with and without the work queues."""
    rng = np.random.default_rng(line)
    for m in (line - 3, line, line + 1):
        sample = np.unique(np.concatenate([[0, 31, 32, 63, 64, 127, 128, m - 130, m - 2, m - 1], rng.integers(0, m, 30)]))
        _attn_case(nq, nkv, hd, C, m + 40, np.arange(40, m + 40), seed=m, sample=sample,
                   n_split="queued" if m != line else None)


@pytest.mark.parametrize("m", [1, 4, 129])
def test_attention_split_8b_context(m):
    """The 8B layer at its full context (32768 cached + 128 prompt tokens):
    the last m rows, as the restore runs them when nothing before the prompt
    is recomputed, with the restore's split choice; every row checked.  One
    and four rows take the few-column kernel (4 and 16 (row, head) columns
    of a KV head), 129 rows the tiled one."""
    w = W.WORKLOADS["8b"]
    mdl = w.model
    S = w.n_ctx + w.n_prompt
    _attn_case(mdl.n_q_heads, mdl.n_kv_heads, mdl.head_dim, mdl.chunk_tokens, S, np.arange(S - m, S), seed=9,
               n_split="auto")
    if m == 4:   # four rows far apart (different splits hold their last keys)
        _attn_case(mdl.n_q_heads, mdl.n_kv_heads, mdl.head_dim, mdl.chunk_tokens, S,
                   np.array([5, 300, 17000, S - 1]), seed=10, n_split="auto")


def test_attention_split_validation():
    torch_cuda()
    with pytest.raises(mz.MzError):
        mz.mz_attention_split(1, 1, 4, 100, 1, 1, 1, 16, 8, 2, 64, 2, 1, 10, 1)   # table short of max_pos
    with pytest.raises(mz.MzError):
        mz.mz_attention_split(1, 1, 4, 10, 1, 1, 1, 16, 8, 2, 64, 2, 1, 10, 1)    # workspace too small
    with pytest.raises(mz.MzError):
        mz.mz_attention_split(1, 1, 4, 10, 1, 1, 1, 16, 8, 2, 64, 65, 1, 1 << 30, 1)   # more than 64 splits
    with pytest.raises(mz.MzError):
        mz.mz_attention_queued(1, 1, 4, 1, 1, 1, 16, 8, 2, 64, 1, 0, 1)   # no work queues
    assert mz.mz_attention_auto_splits(40000, 40000, 32, 8, 128, 64 << 20) == 1   # the chip is full already
    # one decode row (4 columns per KV head): about one workgroup per CU
    assert 24 <= mz.mz_attention_auto_splits(1, 32895, 32, 8, 128, 64 << 20) <= 32
    assert mz.mz_attention_auto_splits(129, 32895, 32, 8, 128, 64 << 20) > 8


@pytest.mark.parametrize("M,d", [(1, 256), (300, 2048), (77, 4096), (5, 1536), (3, 8196), (2, 12292)])
def test_rmsnorm(M, d):
    torch = torch_cuda()
    rng = np.random.default_rng(M * d)
    h = (rng.standard_normal((M, d)) * 3).astype(np.float32)
    h[0, :] *= 1e-3
    x = torch.empty(M, d, device="cuda", dtype=torch.float16)
    dh = torch.from_numpy(h).cuda()
    mz.mz_rmsnorm(dh.data_ptr(), M, d, 1e-5, x.data_ptr(), stream())
    torch.cuda.synchronize()
    ref = O.rmsnorm(h.astype(np.float64), 1e-5)
    got = x.float().cpu().numpy()
    assert np.all(np.abs(got - ref) <= REL * np.abs(ref) + 1e-6)


def test_kernel_entry_validation():
    torch_cuda()
    with pytest.raises(mz.MzError) as e:
        mz.mz_q4_gemm(1, 10, 128, 64, 1, 0, 1)          # n_pad not a multiple of 256
    assert e.value.status == mz.MZ_EINVAL
    with pytest.raises(mz.MzError):
        mz.mz_attention(1, 1, 4, 1, 1, 1, 16, 6, 4, 64, 1)   # 6 q heads over 4 kv heads
    with pytest.raises(mz.MzError):
        mz.mz_attention(1, 1, 4, 1, 1, 8193, 16, 8, 2, 64, 1)   # a chunk table above 8192 entries
    with pytest.raises(mz.MzError):
        mz.mz_attention_split(1, 1, 4, 10, 1, 1, 8193, 16, 8, 2, 64, 2, 1, 1 << 30, 1)


def test_kv_codec_near_code_middles():
    """Values whose quotient lies at or within one half-precision step of the
    middle between two codes, where the kernel forms the correctly rounded
    quotient itself, and groups with infinities: codes and parameters equal
    the oracle's bit for bit.  Steps from subnormal to 2^6, three offsets."""
    from oracle import kv_codec as Q
    torch = torch_cuda()
    rng = np.random.default_rng(3)
    groups = []
    for exp in range(-24, 7):
        for mant in (1.0, 1.25, 1.0 + 2.0 ** -10, 2.0 - 2.0 ** -10, 1.0 + rng.random()):
            d = float(np.float16(mant * 2.0 ** exp))
            for off in (0.0, -100.0 * d, 3.0):
                x = np.concatenate([[0.0, 255.0 * d], (rng.integers(0, 255, 62) + 0.5) * d]) + off
                if np.abs(x).max() >= 65504:
                    continue
                h = x.astype(np.float16)
                h[30:50] = (h[30:50].view(np.uint16) + rng.integers(0, 2, 20).astype(np.uint16)).view(np.float16)
                groups.append(h)
    inf = rng.standard_normal(64).astype(np.float16)
    inf[5], inf[40] = np.inf, -2.0
    groups.append(inf)
    x = np.concatenate(groups)
    n = x.size
    with np.errstate(all="ignore"):
        ref = Q.compress(x)
    d_x = torch.from_numpy(x.view(np.int16)).cuda()
    d_c = torch.empty(Q.compressed_bytes(n), dtype=torch.uint8, device="cuda")
    mz.mz_kv_compress(d_x.data_ptr(), n, d_c.data_ptr(), stream())
    torch.cuda.synchronize()
    got = d_c.cpu().numpy()
    assert np.array_equal(got[:n - 64], ref[:n - 64]), "codes"
    assert np.array_equal(got[n:], ref[n:]), "group parameters"
    assert not got[n - 64:n].any(), "a group of infinite range: every code 0"


@pytest.mark.parametrize("n,scale_kind", [(64, "normal"), (4096, "normal"), (64 * 1237, "mixed"),
                                          (524288, "normal"), (640, "special")])
def test_kv_codec_bit_exact(n, scale_kind):
    """Swap-path codec: codes, per-group (min, step) and reconstruction equal
    the oracle's bit for bit (same fp32 steps, correctly rounded division)."""
    from oracle import kv_codec as Q
    torch = torch_cuda()
    rng = np.random.default_rng(n)
    if scale_kind == "normal":
        x = (rng.standard_normal(n) * 1.7).astype(np.float16)
    elif scale_kind == "mixed":        # per-group scales from 1e-4 to 3e3, offsets
        g = n // 64
        x = (rng.standard_normal((g, 64)) * 10.0 ** rng.uniform(-4, 3.5, (g, 1))
             + rng.uniform(-100, 100, (g, 1))).astype(np.float16).reshape(-1)
    else:                              # constant, two-valued, subnormal, +-0, huge range, ties
        x = np.zeros(n, np.float16)
        x[64:128] = 2.5
        x[128:192] = np.where(np.arange(64) % 2, 1.0, -1.0)
        x[192:256] = np.float16(2.0 ** -20) * np.arange(64)
        x[256:320] = np.where(np.arange(64) % 3 == 0, -0.0, 0.0)
        x[320:384] = np.linspace(-60000, 60000, 64)
        x[384:448] = (np.arange(64) * 0.5 / 16).astype(np.float16)
        x[448:640] = rng.standard_normal(192)
    report("codec", n=n, kind=scale_kind)
    ref = Q.compress(x)
    d_x = torch.from_numpy(x.view(np.int16)).cuda()
    d_c = torch.empty(Q.compressed_bytes(n), dtype=torch.uint8, device="cuda")
    d_y = torch.empty(n, dtype=torch.int16, device="cuda")
    mz.mz_kv_compress(d_x.data_ptr(), n, d_c.data_ptr(), stream())
    mz.mz_kv_decompress(d_c.data_ptr(), n, d_y.data_ptr(), stream())
    torch.cuda.synchronize()
    got = d_c.cpu().numpy()
    assert np.array_equal(got[:n], ref[:n]), "codes"
    assert np.array_equal(got[n:], ref[n:]), "group parameters"
    assert np.array_equal(d_y.cpu().numpy().view(np.float16).view(np.uint16),
                          Q.decompress(ref, n).view(np.uint16)), "reconstruction"
