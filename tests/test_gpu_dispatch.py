"""Edges of the size rules that choose between kernels and launch shapes, through
the C ABI at the repository's tolerances: the attention and the cache's codes
against the CPU oracle, the products and the controller against plain torch in
fp32 or fp64 on the same operands, the lists and the chunk counts against the
same work done by another route on the device."""
import numpy as np
import pytest
import torch

import gen
import oracle
import paper_2607_06601_amd as tr
from paper_2607_06601_amd.device import DeviceLayer, to_dev

from _common import assert_close, bound_of, note, npy, torch_act

pytestmark = pytest.mark.gpu
DEV = "cuda"


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    tr.lib()
    yield
    torch.cuda.synchronize()


def _append(c, cache, b, k, v, bits, act):
    n = len(bits)
    tr.kv_append(c, cache, 1, n, to_dev(k.reshape(n, -1), torch_act(act)),
                 to_dev(v.reshape(n, -1), torch_act(act)), to_dev(bits, torch.uint8),
                 tr.workspace(c, tr.OP_KV_APPEND, 1, n),
                 seq_ids=torch.tensor([b], dtype=torch.int32, device=DEV))


@pytest.mark.parametrize("B,H,Hkv,dh,cap,lens", [
    (1, 1, 1, 128, 17000, [17000]),          # the most chunks (32), 8 in flight at a time
    (1, 4, 1, 64, 1088, [1000]),             # 17 tiles: one chunk, no combine
    (1, 4, 1, 64, 1089, [1089]),             # 18 tiles: three chunks
    (3, 4, 2, 128, 9000, [9000, 1, 33]),     # chunks without a key beside full ones
    (5, 6, 3, 64, 20000, [5000, 64, 1, 999, 4097]),  # 15 pairs: 17 chunks
    (16, 2, 1, 64, 20000, [2000] * 8 + [1, 2, 15, 16, 17, 63, 64, 65]),  # 16 pairs: 16 chunks
])
def test_decode_chunk_counts(B, H, Hkv, dh, cap, lens):
    w, act = 100, "bf16"
    c = tr.make_cfg(256, H, Hkv, dh, w, 4, 1, 512, 64, act)
    cache = tr.KVCache(c, B, cap)
    rng = gen.stream(31, "chunks", B, cap)
    modes = rng.choice(3, size=(B, H), p=[0.1, 0.3, 0.6]).astype(np.uint8)
    modes[:, 0] = 2
    q = gen.to_act(gen.normal(31, "chunk_q", (B, H, dh), 0.8), act)
    kv = {}
    for b, n in enumerate(lens):
        k, v = gen.kv_block(31 + b, n, Hkv, dh, act, 0.8)
        bits = rng.integers(0, 4, n).astype(np.uint8)
        kv[b] = (k, v, bits)
        _append(c, cache, b, k, v, bits, act)
    assert cache.status() == 0
    o = torch.empty(B, H * dh, dtype=torch_act(act), device=DEV)
    tr.attn_decode(c, B, to_dev(q.reshape(B, -1), torch_act(act)), cache,
                   to_dev(modes, torch.uint8), o, ws=tr.workspace(c, tr.OP_ATTN_DECODE, B, 1))
    torch.cuda.synchronize()
    og = npy(o).reshape(B, H, dh)
    for b, n in enumerate(lens):
        khat, vhat, _ = oracle.layer.store_kv(*kv[b], dict(G=64))
        ref = oracle.attention_seq(np.asarray(q[b:b + 1], np.float64), np.array([n - 1]), khat,
                                   vhat, modes[b:b + 1], w)[0]
        assert_close(og[b], ref, act, f"o[b={b}]")


def _small_layer(monkeypatch, **shape):
    """A layer of a small shape of its own (uncalibrated routing: every option occurs)."""
    cfg = dict(kind="prefill", d=256, E=4, k=2, d_ff=2048, G=64, act="bf16", seeds=(7,),
               modes=(0.3, 0.4, 0.3), bits=(0.25, 0.25, 0.25, 0.25), experts="uniform")
    cfg.update(shape)
    monkeypatch.setitem(gen.CONFIGS, "small", cfg)
    return gen.make_layer("small", 7)


@pytest.mark.parametrize("B,T,H,Hkv,dh,w,ctx,pages", [
    (1, 1, 4, 1, 64, 100, 3000, None),       # one query tile, full mode split, local not
    (2, 17, 4, 2, 128, 600, 2500, None),     # both modes split, a ragged second query tile
    (1, 64, 6, 3, 64, 1000, 700, 2),         # paged; windows longer than some ranges
    (3, 33, 8, 1, 64, 300, 0, None),         # two quartets
    (1, 700, 8, 1, 64, 300, 0, None),        # chunks without a key (early queries of a prompt)
    (1, 400, 4, 4, 128, 256, 1100, None),    # one head per kv head
])
def test_prefill_split_key_ranges(monkeypatch, B, T, H, Hkv, dh, w, ctx, pages):
    """The layer's attention (key ranges split over its scratch) against the
    stage call (never split) on the same queries, modes and cache: both round
    the same sums, taken in another order, to bf16.  Then against the oracle's
    attention over the same cached keys and values."""
    L = _small_layer(monkeypatch, B=B, T=T, H=H, Hkv=Hkv, dh=dh, w=w)
    D = DeviceLayer(L)
    c, N = D.cfg, B * T
    n_seq, cap = B + 2, 20000 if ctx else 4096
    pg = None if pages is None else (pages, [64] * 4)
    cache = tr.KVCache(c, n_seq, cap, pages=pg)
    rng = gen.stream(41, "split", T, ctx)
    ids, held = list(rng.permutation(n_seq)[:B]), {}
    if ctx:
        for s in ids:
            n = int(ctx * (0.5 + 0.5 * rng.random()))
            k, v = gen.kv_block(41 + int(s), n, Hkv, dh, "bf16", 0.8)
            held[s] = (k, v, rng.integers(0, 4, n).astype(np.uint8))
            _append(c, cache, int(s), *held[s], "bf16")
    if B > 2:
        ids[1] = n_seq                           # a row outside the cache: zeros
    sid = torch.tensor([int(s) for s in ids], dtype=torch.int32, device=DEV)
    t = dict(q=torch.empty(N, H * dh, dtype=D.act, device=DEV),
             o=torch.full((N, H * dh), float("nan"), dtype=D.act, device=DEV),
             mode=torch.empty(N, H, dtype=torch.uint8, device=DEV),
             k=torch.empty(N, Hkv * dh, dtype=D.act, device=DEV),
             v=torch.empty(N, Hkv * dh, dtype=D.act, device=DEV),
             bit=torch.empty(N, dtype=torch.uint8, device=DEV))
    x_out = torch.empty(N, L["cfg"]["d"], dtype=D.act, device=DEV)
    ws = tr.workspace(c, tr.OP_LAYER_PREFILL, B, T)
    ws.fill_(0xFF)                               # scratch holds NaNs
    print(f"split prefill B={B} T={T} H={H}/{Hkv} dh={dh} ctx={ctx}", flush=True)
    tr.layer_prefill(c, B, T, D.x, D.psi, D.rw, D.dw, D.mw, cache, x_out, ws,
                     taps=tr.Taps(**{n: v.data_ptr() for n, v in t.items()}), seq_ids=sid)
    torch.cuda.synchronize()
    cmp = tr.CompactionBuffers(c, B, T)
    n1, bit = torch.empty_like(x_out), torch.empty(N, dtype=torch.uint8, device=DEV)
    mode = torch.empty_like(t["mode"])
    eidx = torch.empty(N, 2, dtype=torch.int32, device=DEV)
    tr.router(c, B, T, D.x, D.psi, D.rw, n1, mode, bit, eidx,
              torch.empty(N, 2, device=DEV), cmp.struct, tr.workspace(c, tr.OP_ROUTER, B, T))
    assert torch.equal(mode, t["mode"])
    o = torch.empty_like(t["o"])
    tr.attn_prefill(c, B, T, t["q"], cache, mode, cmp.struct, o, seq_ids=sid)
    torch.cuda.synchronize()
    assert {0, 1, 2} == set(npy(mode).ravel().tolist()) or N < 8
    assert_close(npy(t["o"]), npy(o), "bf16", "o (split against unsplit)")
    if B > 2:
        assert not npy(t["o"]).reshape(B, -1)[1].any()
    r = {n: npy(v).reshape(B, T, *v.shape[1:]) for n, v in t.items()}
    for b, s in enumerate(ids):
        if s == n_seq:
            continue
        k, v = (r[n][b].reshape(T, Hkv, dh) for n in "kv")
        bits = r["bit"][b]
        if s in held:
            k, v, bits = (np.concatenate(p) for p in zip(held[s], (k, v, bits)))
        khat, vhat, _ = oracle.layer.store_kv(k, v, bits, dict(G=64))
        ref = oracle.attention_seq(r["q"][b].reshape(T, H, dh).astype(np.float64),
                                   np.arange(len(bits) - T, len(bits)), khat, vhat, r["mode"][b], w)
        assert_close(r["o"][b], ref.reshape(T, -1), "bf16", f"o[{b}] (against the oracle)")


@pytest.mark.parametrize("act,T,len0,layer", [
    ("bf16", 1500, 700, True),      # key ranges split: 800 queries before the first key
    ("bf16", 40, 37, True),         # unsplit; a query tile on both sides of position 0
    ("bf16", 1500, 700, False), ("f32", 300, 70, True), ("f32", 300, 70, False),
])
def test_prefill_of_a_dropped_row(monkeypatch, act, T, len0, layer):
    """A row dropped for its length (len0 + T tokens past the capacity) whose
    first queries would lie before the sequence's first position: they have no
    key, so their attention is zero (not what the scratch or o held); the other
    queries of the row see the keys that are there, and the row beside it is
    as without it."""
    H, Hkv, dh, w = 4, 2, 64, 400
    L = _small_layer(monkeypatch, B=2, T=T, H=H, Hkv=Hkv, dh=dh, w=w, act=act)
    D = DeviceLayer(L)
    c, N = D.cfg, 2 * T
    rng = gen.stream(43, "dropped", T, len0)
    kv = gen.kv_block(43, len0, Hkv, dh, act, 0.8)
    bits = rng.integers(0, 4, len0).astype(np.uint8)
    out = []
    for dropped in (True, False):
        cache = tr.KVCache(c, 2, T + len0 - dropped)
        _append(c, cache, 0, *kv, bits, act)
        t = {n: torch.full((N, m), float("nan"), dtype=D.act, device=DEV)
             for n, m in (("q", H * dh), ("o", H * dh), ("xt", 256))}
        t["mode"] = torch.full((N, H), 9, dtype=torch.uint8, device=DEV)
        x_out = torch.full((N, 256), float("nan"), dtype=D.act, device=DEV)
        ws = tr.workspace(c, tr.OP_LAYER_PREFILL, 2, T)
        ws.fill_(0xFF)                           # scratch holds NaNs
        print(f"dropped row act={act} T={T} len0={len0} layer={layer} {dropped}", flush=True)
        tr.layer_prefill(c, 2, T, D.x, D.psi, D.rw, D.dw, D.mw, cache, x_out, ws,
                         taps=tr.Taps(**{n: v.data_ptr() for n, v in t.items()}))
        assert cache.status() == (tr.CACHE_OVERFLOW if dropped else 0)
        if not layer:
            cmp = tr.CompactionBuffers(c, 2, T)
            cc = oracle.compact(npy(t["mode"]), np.zeros((N, 1), np.int32), 2, T, H, 4, 1)
            cmp.attn_cnt.copy_(torch.from_numpy(cc["attn_cnt"]))
            cmp.attn_idx.copy_(torch.from_numpy(np.maximum(cc["attn_idx"], 0).reshape(-1)))
            t["o"].fill_(float("nan"))
            tr.attn_prefill(c, 2, T, t["q"], cache, t["mode"], cmp.struct, t["o"])
        torch.cuda.synchronize()
        out.append(dict({n: npy(v).reshape(2, T, -1) for n, v in t.items()}, x_out=npy(x_out)))
    got, whole = out
    neg = T - len0                               # queries at positions < 0
    assert not got["o"][0, :neg].any()
    pos = np.arange(neg, T) - neg
    khat, vhat, _ = oracle.layer.store_kv(*kv, bits, dict(G=64))
    ref = oracle.attention_seq(got["q"][0, neg:].reshape(-1, H, dh).astype(np.float64), pos, khat,
                               vhat, got["mode"][0, neg:], w)
    assert_close(got["o"][0, neg:], ref.reshape(len(pos), -1), act, "o of the dropped row")
    np.testing.assert_array_equal(got["o"][1], whole["o"][1])
    assert np.isfinite(got["x_out"]).all()


@pytest.mark.parametrize("B,T,H,Hkv,dh,w,lens", [
    (1, 333, 16, 4, 64, 256, [0]),               # one chunk, two, and several
    (2, 300, 4, 2, 128, 600, [0, 400]), (1, 64, 4, 1, 64, 900, [4000]),
])
def test_chunks_follow_the_content(monkeypatch, B, T, H, Hkv, dh, w, lens):
    """The chunks of a key range follow the keys that are cached, not the room
    in the cache: the same bits from a cache that is full after the call and
    from one of 32768 positions."""
    L = _small_layer(monkeypatch, B=B, T=T, H=H, Hkv=Hkv, dh=dh, w=w)
    D = DeviceLayer(L)
    c, N = D.cfg, B * T
    res = []
    for cap in (max(lens) + T, 32768):
        cache = tr.KVCache(c, B, cap)
        rng = gen.stream(44, "room", T, lens[0])
        for b, n in enumerate(lens):
            if n:
                k, v = gen.kv_block(44 + b, n, Hkv, dh, "bf16", 0.8)
                _append(c, cache, b, k, v, rng.integers(0, 4, n).astype(np.uint8), "bf16")
        o = torch.full((N, H * dh), float("nan"), dtype=D.act, device=DEV)
        x_out = torch.empty(N, 256, dtype=D.act, device=DEV)
        taps = tr.Taps(o=o.data_ptr())
        ws = tr.workspace(c, tr.OP_LAYER_PREFILL, B, T)
        ws.fill_(0xFF)
        print(f"content B={B} T={T} lens={lens} cap={cap}", flush=True)
        tr.layer_prefill(c, B, T, D.x, D.psi, D.rw, D.dw, D.mw, cache, x_out, ws, taps=taps)
        assert cache.status() == 0
        res.append((npy(o), npy(x_out)))
    for a, b in zip(*res):
        np.testing.assert_array_equal(a, b)


@pytest.mark.parametrize("H,Hkv,dh", [(4, 2, 64), (8, 1, 128)])  # heads packed, a head a column
def test_decode_chunks_of_a_mixed_batch(H, Hkv, dh):
    """Long, short and empty rows and one outside the cache in one launch of
    many chunks, most of them without a key in the short rows, over scratch that
    holds NaNs: each row against the oracle."""
    lens, ids, act, w = [3000, 40, 0, 1500, 0], [0, 1, 2, 9, 3], "bf16", 200
    c = tr.make_cfg(256, H, Hkv, dh, w, 4, 1, 512, 64, act)
    B = len(ids)
    rng = gen.stream(45, "mixed", H)
    modes = rng.choice(3, size=(B, H), p=[0.1, 0.3, 0.6]).astype(np.uint8)
    q = gen.to_act(gen.normal(45, "mixed_q", (B, H, dh), 0.8), act)
    cache, kv = tr.KVCache(c, len(lens), 20000), {}
    for s, n in enumerate(lens):
        if n:
            k, v = gen.kv_block(45 + s, n, Hkv, dh, act, 0.8)
            kv[s] = (k, v, rng.integers(0, 4, n).astype(np.uint8))
            _append(c, cache, s, *kv[s], act)
    o = torch.full((B, H * dh), float("nan"), dtype=torch_act(act), device=DEV)
    ws = tr.workspace(c, tr.OP_ATTN_DECODE, B, 1)
    ws.fill_(0xFF)
    tr.attn_decode(c, B, to_dev(q.reshape(B, -1), torch_act(act)), cache, to_dev(modes, torch.uint8),
                   o, ws=ws, seq_ids=torch.tensor(ids, dtype=torch.int32, device=DEV))
    og = npy(o).reshape(B, H, dh)
    for r, s in enumerate(ids):
        if s not in kv:
            assert not og[r].any()
            continue
        khat, vhat, _ = oracle.layer.store_kv(*kv[s], dict(G=64))
        ref = oracle.attention_seq(np.asarray(q[r:r + 1], np.float64), np.array([lens[s] - 1]), khat,
                                   vhat, modes[r:r + 1], w)[0]
        assert_close(og[r], ref, act, f"o[{r}]")


# ------------------------------------------------------- GEMM tile choices
@pytest.mark.parametrize("H,Hkv,dh,d,n_tok", [
    (4, 1, 64, 128, 1), (3, 1, 64, 128, 33),           # O-projection: two K groups (K 192: one)
    (12, 2, 64, 1024, 512), (12, 2, 64, 1024, 513),    # 256 blocks of them and more
    (4, 1, 64, 256, 4032), (4, 1, 64, 256, 4033),      # 32-row tiles to 64 x 128 (3 columns of 128)
    (3, 1, 64, 192, 6200),                             # 320 columns: the last tile half empty
    (16, 4, 128, 128, 768), (16, 4, 128, 128, 769),    # 288 tiles of 64 rows; 128 x 128, one round
    (16, 4, 128, 128, 1280), (16, 4, 128, 128, 1281),  # its last; 64 x 128, three blocks a CU
    (16, 4, 128, 128, 2049), (16, 4, 128, 128, 2700),  # 128 x 128, two a CU; 256 x 256, four waves
    (16, 8, 64, 128, 4000),                            # 256 x 128, four waves
])
def test_projection_tiles(H, Hkv, dh, d, n_tok):
    """QKV and the O-projection on both sides of their tile choices, against
    plain fp32 products of the same bf16 operands."""
    c = tr.make_cfg(d, H, Hkv, dh, 64, 4, 1, 512, 64, "bf16")
    g = torch.Generator(device=DEV)
    g.manual_seed(51)

    def rnd(*shape, std=1.0):
        return (torch.randn(shape, generator=g, device=DEV) * std).bfloat16()

    nq, nkv = H * dh, Hkv * dh
    w, wo, n1, x = rnd(nq + 2 * nkv, d, std=d ** -0.5), rnd(d, nq, std=nq ** -0.5), rnd(n_tok, d), \
        rnd(n_tok, d)
    dw = tr.DenseW(Wq=w.data_ptr(), Wk=w[nq:].data_ptr(), Wv=w[nq + nkv:].data_ptr(),
                   Wo=wo.data_ptr())
    out = {n: torch.full((n_tok, m), float("nan"), dtype=torch.bfloat16, device=DEV)
           for n, m in (("q", nq), ("k", nkv), ("v", nkv))}
    xt = torch.full((n_tok, d), float("nan"), dtype=torch.bfloat16, device=DEV)
    print(f"projections H={H}/{Hkv} dh={dh} d={d} n={n_tok}", flush=True)
    tr.qkv(c, 1, n_tok, n1, dw, out["q"], out["k"], out["v"],
           tr.workspace(c, tr.OP_QKV, 1, n_tok))
    tr.oproj(c, n_tok, x, out["q"], dw, xt)
    torch.cuda.synchronize()
    y = n1.float() @ w.float().t()
    half = dh // 2
    inv = 1e4 ** (-2.0 * torch.arange(half, dtype=torch.float64, device=DEV) / dh)
    ang = torch.arange(n_tok, dtype=torch.float64, device=DEV)[:, None, None] * inv
    cs, sn = ang.cos().float(), ang.sin().float()

    def rope(t):
        t = t.reshape(n_tok, -1, dh)
        a, b = t[..., :half], t[..., half:]
        return torch.cat([a * cs - b * sn, a * sn + b * cs], -1).reshape(n_tok, -1)

    ref = dict(q=rope(y[:, :nq]), k=rope(y[:, nq:nq + nkv]), v=y[:, nq + nkv:])
    for n, t in out.items():
        assert_close(npy(t), npy(ref[n]), "bf16", n)
    assert_close(npy(xt), npy(x.float() + out["q"].float() @ wo.float().t()), "bf16", "xt")


@pytest.mark.parametrize("E,k,d,dff,n_tok,skew", [
    (4, 1, 256, 512, 1, 0), (8, 2, 2048, 4096, 4, 0),     # fewer assignments than experts: K groups
    (8, 2, 2048, 384, 60, 0), (8, 2, 2048, 384, 100, 1),  # long K: K groups in gate/up
    (4, 1, 256, 512, 124, 0), (4, 1, 256, 512, 125, 0),   # 24 rows an expert and one more
    (4, 1, 256, 512, 324, 0), (4, 1, 256, 512, 325, 0),   # 64 and 65
    (16, 2, 1024, 256, 300, 0),                           # down: 64 x 128 over K halves
    (4, 2, 2048, 256, 700, 0),                            # down: 128 x 128 over K halves
    (8, 2, 256, 4096, 900, 0),                            # gate/up: four waves, 128 rows
    (4, 2, 256, 512, 1024, 0), (4, 2, 256, 512, 1025, 0), # K halves end; 128 x 128 down tiles
    (8, 2, 1024, 2048, 3000, 0),                          # 128-row four-wave tiles in both
    (8, 2, 768, 320, 3001, 0),                            # d a multiple of 192 and 256
    (16, 2, 2048, 192, 2000, 0),                          # one 256-row tile an expert
    (3, 2, 192, 192, 4000, 0), (3, 2, 192, 192, 40000, 0),  # 192-wide columns only
    (2, 1, 64, 64, 3000, 0),                              # K too short for the four-wave kernel
    (8, 2, 512, 384, 2100, 1), (8, 2, 512, 384, 150, 1),  # one expert takes nearly all rows
])
def test_expert_tiles(E, k, d, dff, n_tok, skew):
    """The expert block on both sides of its tile choices, against fp32 torch
    (n2 and the SwiGLU product held in bf16, as the layer's contract has them)."""
    c = tr.make_cfg(d, 4, 1, 64, 64, E, k, dff, 64, "bf16")
    g = torch.Generator(device=DEV)
    g.manual_seed(52)

    def rnd(*shape, std=1.0):
        return (torch.randn(shape, generator=g, device=DEV) * std).bfloat16()

    xt, g2 = rnd(n_tok, d), rnd(d, std=0.02) + 1
    wg, wu, wd = rnd(E, dff, d, std=d ** -0.5), rnd(E, dff, d, std=d ** -0.5), rnd(E, d, dff,
                                                                                  std=dff ** -0.5)
    z = torch.randn(n_tok, E + 1, generator=g, device=DEV)
    if skew:
        z[:, 2] += 6
    eidx = z.topk(k).indices.sort(1).values
    gate = torch.softmax(torch.randn(n_tok, k, generator=g, device=DEV), 1)
    cmp = tr.CompactionBuffers(c, 1, n_tok)
    cnt = torch.bincount(eidx.reshape(-1), minlength=E + 1)
    cmp.exp_cnt.copy_(cnt)
    cmp.exp_off[1:].copy_(cnt[1:].cumsum(0))
    cmp.exp_rows[:n_tok * k - int(cnt[0])].copy_(
        eidx.reshape(-1).argsort(stable=True)[int(cnt[0]):])
    x_out = torch.full_like(xt, float("nan"))
    ws = tr.workspace(c, tr.OP_MOE, n_tok, 1)
    ws.fill_(0xFF)
    print(f"experts E={E} k={k} d={d} dff={dff} n={n_tok}", flush=True)
    tr.moe(c, n_tok, xt, tr.DenseW(g2=g2.data_ptr()),
           tr.MoeW(wg.data_ptr(), wu.data_ptr(), wd.data_ptr()), eidx.int().contiguous(), gate,
           cmp.struct, x_out, ws)
    torch.cuda.synchronize()
    xd = xt.double()
    n2 = (xd * torch.rsqrt(xd.square().mean(1, keepdim=True) + 1e-6) * g2.double()).bfloat16()
    ref, flip = xt.float().clone(), torch.zeros(n_tok, device=DEV)
    for e in range(1, E + 1):
        rows, slot = (eidx == e).nonzero(as_tuple=True)
        u = n2[rows].float()
        h = torch.nn.functional.silu(u @ wg[e - 1].float().t()) * (u @ wu[e - 1].float().t())
        ref.index_add_(0, rows, (h.bfloat16().float() @ wd[e - 1].float().t())
                       * gate[rows, slot][:, None])
        # the two sides' fp32 sums differ in their last bits, and where that
        # moves an element of H to the next bf16 value (2^-8 of it at most)
        # the row's outputs move by that much times a weight and the gate;
        # more than one of the largest elements of a row does not
        flip.index_add_(0, rows, h.abs().amax(1) * gate[rows, slot] * wd[e - 1].abs().amax() / 256)
    err = np.abs(npy(x_out).astype(np.float64) - npy(ref))
    ratio = float((err / (bound_of(npy(ref), "bf16") + npy(flip)[:, None])).max())
    note("x_out (one H step allowed)", ratio)
    assert ratio <= 1.0, ratio


# --------------------------------------------------------------- fp32 path
@pytest.mark.parametrize("H,Hkv,dh,d,dff,E,k,n_tok", [
    (4, 1, 64, 64, 64, 2, 1, 1),        # K 64 split over four waves, one row
    (2, 1, 128, 192, 320, 3, 2, 33),    # an odd number of 32-column units, a ragged row tile
    (8, 2, 128, 512, 1024, 4, 2, 2111), # 64 x 64 tiles over all of K
    (3, 1, 64, 448, 192, 5, 5, 2900),   # the same with an odd number of units
])
def test_f32_products(H, Hkv, dh, d, dff, E, k, n_tok):
    """fp32 projections and experts against fp64 torch, within the fp32 bound
    1e-5 (|ref| + rms(ref))."""
    c = tr.make_cfg(d, H, Hkv, dh, 64, E, k, dff, 32, "f32")
    g = torch.Generator(device=DEV)
    g.manual_seed(61)

    def rnd(*shape, std=1.0):
        return torch.randn(shape, generator=g, device=DEV) * std

    nq, nkv = H * dh, Hkv * dh
    w, wo, n1, x = rnd(nq + 2 * nkv, d, std=d ** -0.5), rnd(d, nq, std=nq ** -0.5), rnd(n_tok, d), \
        rnd(n_tok, d)
    g2, wg, wu = rnd(d, std=0.02) + 1, rnd(E, dff, d, std=d ** -0.5), rnd(E, dff, d, std=d ** -0.5)
    wd = rnd(E, d, dff, std=dff ** -0.5)
    dw = tr.DenseW(Wq=w.data_ptr(), Wk=w[nq:].data_ptr(), Wv=w[nq + nkv:].data_ptr(),
                   Wo=wo.data_ptr(), g2=g2.data_ptr())
    out = {n: torch.full((n_tok, m), float("nan"), device=DEV)
           for n, m in (("q", nq), ("k", nkv), ("v", nkv), ("xt", d), ("x_out", d))}
    print(f"f32 products d={d} n={n_tok}", flush=True)
    tr.qkv(c, 1, n_tok, n1, dw, out["q"], out["k"], out["v"], tr.workspace(c, tr.OP_QKV, 1, n_tok))
    tr.oproj(c, n_tok, x, out["q"], dw, out["xt"])
    eidx = torch.randn(n_tok, E + 1, generator=g, device=DEV).topk(k).indices.sort(1).values
    gate = torch.softmax(torch.randn(n_tok, k, generator=g, device=DEV), 1)
    cmp = tr.CompactionBuffers(c, 1, n_tok)
    cnt = torch.bincount(eidx.reshape(-1), minlength=E + 1)
    cmp.exp_cnt.copy_(cnt)
    cmp.exp_off[1:].copy_(cnt[1:].cumsum(0))
    cmp.exp_rows[:n_tok * k - int(cnt[0])].copy_(
        eidx.reshape(-1).argsort(stable=True)[int(cnt[0]):])
    tr.moe(c, n_tok, x, dw, tr.MoeW(wg.data_ptr(), wu.data_ptr(), wd.data_ptr()),
           eidx.int().contiguous(), gate, cmp.struct, out["x_out"], tr.workspace(c, tr.OP_MOE, n_tok, 1))
    torch.cuda.synchronize()
    y = n1.double() @ w.double().t()
    half = dh // 2
    inv = 1e4 ** (-2.0 * torch.arange(half, dtype=torch.float64, device=DEV) / dh)
    ang = torch.arange(n_tok, dtype=torch.float64, device=DEV)[:, None, None] * inv

    def rope(t):
        t = t.reshape(n_tok, -1, dh)
        a, b = t[..., :half], t[..., half:]
        return torch.cat([a * ang.cos() - b * ang.sin(), a * ang.sin() + b * ang.cos()],
                         -1).reshape(n_tok, -1)

    xd = x.double()
    ref = dict(q=rope(y[:, :nq]), k=rope(y[:, nq:nq + nkv]), v=y[:, nq + nkv:],
               xt=xd + out["q"].double() @ wo.double().t(), x_out=xd.clone())
    n2 = xd * torch.rsqrt(xd.square().mean(1, keepdim=True) + 1e-6) * g2.double()
    for e in range(1, E + 1):
        rows, slot = (eidx == e).nonzero(as_tuple=True)
        u = n2[rows]
        h = torch.nn.functional.silu(u @ wg[e - 1].double().t()) * (u @ wu[e - 1].double().t())
        ref["x_out"].index_add_(0, rows, (h @ wd[e - 1].double().t())
                                * gate[rows, slot].double()[:, None])
    for n, t in out.items():
        assert_close(npy(t), npy(ref[n]), "f32", n)


@pytest.mark.parametrize("H,Hkv,dh,G,w,lens", [
    (2, 1, 64, 64, 50, [1, 63, 64, 65, 700]), (4, 2, 64, 32, 1000, [300, 31]),
    (3, 1, 128, 32, 40, [500, 33, 1]), (2, 2, 128, 64, 200, [161]),
])
def test_f32_attention(H, Hkv, dh, G, w, lens):
    """fp32 attention, decode and prefill of the last 5 tokens, over every
    width; slots past a pool's length hold infinities."""
    B, act, T = len(lens), "f32", 5
    c = tr.make_cfg(256, H, Hkv, dh, w, 4, 1, 512, G, act)
    cache = tr.KVCache(c, B, max(lens) + T)
    rng = gen.stream(62, "f32attn", dh, G)
    kv = {}
    for b, n in enumerate(lens):
        n += T
        k, v = gen.kv_block(62 + b, n, Hkv, dh, act, 0.8)
        bits = rng.integers(0, 4, n).astype(np.uint8)
        kv[b] = (k, v, bits)
        bad = np.full((40, Hkv, dh), np.inf, np.float32)     # left behind by an earlier sequence
        if n > 40:
            _append(c, cache, b, bad, bad, np.full(40, 3, np.uint8), act)
            cache.reset_seq(b)
        _append(c, cache, b, k, v, bits, act)
    assert cache.status() == 0
    q = gen.normal(62, "f32_q", (B, T, H, dh), 0.8)
    modes = rng.choice(3, size=(B, T, H), p=[0.1, 0.45, 0.45]).astype(np.uint8)
    modes[:, -1, 0] = 2
    modes[:, -1, -1] = 1
    od, op = torch.empty(B, H * dh, device=DEV), torch.empty(B * T, H * dh, device=DEV)
    tr.attn_decode(c, B, to_dev(q[:, -1].reshape(B, -1), torch.float32), cache,
                   to_dev(modes[:, -1], torch.uint8), od, ws=tr.workspace(c, tr.OP_ATTN_DECODE, B, 1))
    cmp = tr.CompactionBuffers(c, B, T)
    cc = oracle.compact(modes.reshape(B * T, H), np.zeros((B * T, 1), np.int32), B, T, H, 4, 1)
    cmp.attn_cnt.copy_(torch.from_numpy(cc["attn_cnt"]))
    cmp.attn_idx.copy_(torch.from_numpy(np.maximum(cc["attn_idx"], 0).reshape(-1)))
    tr.attn_prefill(c, B, T, to_dev(q.reshape(B * T, -1), torch.float32), cache,
                    to_dev(modes.reshape(B * T, H), torch.uint8), cmp.struct, op)
    torch.cuda.synchronize()
    for b, n in enumerate(lens):
        khat, vhat, _ = oracle.layer.store_kv(*kv[b], dict(G=G))
        ref = oracle.attention_seq(q[b].astype(np.float64), np.arange(n, n + T), khat, vhat,
                                   modes[b], w)
        assert_close(npy(op).reshape(B, T, H, dh)[b], ref, act, f"prefill o[b={b}]")
        assert_close(npy(od).reshape(B, H, dh)[b], ref[-1], act, f"decode o[b={b}]")


# --------------------------------------------------- controller's backward
@pytest.mark.parametrize("B,T,d,dpsi,H,E,k,groups,act,big", [
    (1, 1, 64, 0, 2, 1, 1, 0, "bf16", 0),       # one token, one column tile, no side features
    (1, 31, 128, 4, 4, 3, 2, 2, "f32", 0),      # fewer tokens than a tile
    (2, 67, 192, 32, 4, 2, 3, 1, "bf16", 0),    # a ragged wave of tokens, the most side features
    (1, 129, 2048, 8, 16, 16, 2, 0, "bf16", 0), # one token past a block, many column tiles
    (3, 683, 64, 8, 30, 12, 2, 0, "f32", 0),    # 107 logits; several chunks, few column tiles
    (1, 300, 64, 8, 4, 3, 2, 0, "f32", 1000),   # biases and side features far above W1 n1:
    (1, 33, 64, 0, 4, 3, 2, 0, "bf16", 1000),   # psi in a chunk of K of its own; no psi;
    (1, 9000, 320, 32, 4, 3, 2, 0, "f32", 1000),  # three chunks of x and one of both
])
def test_relaxed_backward_tiles(B, T, d, dpsi, H, E, k, groups, act, big):
    """Gradients of the relaxed controller against fp64 torch autograd at the
    edges of the token, column and chunk tiles, within the fp32 bound (the
    sums run over at most 9000 tokens).  big: trunk biases and side features of
    that size, whose share of a1 is not to cost dx the bits of W1 n1 (they
    saturate the GELU, so that the rounding of a1 itself moves nothing)."""
    A, N, dev = groups or H, B * T, dict(device=DEV)
    c = tr.make_cfg(d, H, 2, 64, 64, E, k, 128, 64, act, d_psi=dpsi, attn_groups=groups)
    g = torch.Generator(**dev)
    g.manual_seed(71)

    def rnd(*shape, std=1.0):
        return torch.randn(shape, generator=g, **dev) * std

    w = dict(g1=1 + rnd(d, std=0.02), W1=rnd(128, d + dpsi, std=0.05), b1=rnd(128, std=0.02),
             W2=rnd(128, 128, std=0.1), b2=rnd(128, std=0.02), gr=1 + rnd(128, std=0.02),
             Wa=rnd(3 * A, 128, std=0.1), ca=rnd(3 * A, std=0.1), We=rnd(E + 1, 128, std=0.1),
             ce=rnd(E + 1, std=0.1), Wb=rnd(4, 128, std=0.1), cb=rnd(4, std=0.1))
    if big:
        w["b1"] = big * (2 + torch.rand(128, generator=g, **dev)) * rnd(128).sign()
    rw = tr.RouterW(*(t.data_ptr() for t in w.values()))
    x, psi = rnd(N, d).to(torch_act(act)), rnd(N, max(dpsi, 1))[:, :dpsi].contiguous()
    psi *= big or 1
    pos = torch.arange(N, dtype=torch.int32, **dev)
    ga, gb = rnd(N, A, 3), rnd(N, 4)
    p = tr.RelaxParams(g_attn=ga.data_ptr(), g_bits=gb.data_ptr(), pos=pos.data_ptr(), tau_a=1.3,
                       tau_b=0.8, zeta=0.99, alpha=0.01, beta=0.001, gamma=0.1)
    f64, dec = dict(dtype=torch.float64, **dev), {}
    o = dict(y_attn=torch.empty(N, A, 3, **dev), y_bits=torch.empty(N, 4, **dev),
             c_flops=torch.empty(N, **dev), c_mem=torch.empty(N, **dev),
             stats=torch.empty(tr.RELAX_NSTAT, **f64), usage_exp=torch.empty(2, E + 1, **f64))
    fwd = tr.RelaxOut(**{n: t.data_ptr() for n, t in o.items()})
    eidx, egate = torch.empty(N, k, dtype=torch.int32, **dev), torch.empty(N, k, **dev)
    cmp = tr.CompactionBuffers(c, B, T)
    tr.router_relaxed(c, B, T, x, psi, rw, p, torch.empty_like(x),
                      torch.empty(N, H, dtype=torch.uint8, **dev),
                      torch.empty(N, dtype=torch.uint8, **dev), eidx, egate, cmp.struct, fwd,
                      tr.workspace(c, tr.OP_ROUTER_RELAXED, B, T))
    up = dict(a=rnd(N, A, 3), b=rnd(N, 4), e=rnd(N, k))
    rho = torch.tensor([1.5, 0.8, 2.5], **f64)
    gin = tr.RelaxGradIn(g_attn=up["a"].data_ptr(), g_bits=up["b"].data_ptr(),
                         g_gate=up["e"].data_ptr(), rho=rho.data_ptr(), rho_m=0.0)
    out = {"d" + n: torch.full_like(t, float("nan")) for n, t in w.items()}
    out.update(dx=torch.full((N, d), float("nan"), **dev), dpsi=torch.full((N, dpsi), float("nan"), **dev))
    ws = tr.workspace(c, tr.OP_ROUTER_RELAXED_BACKWARD, B, T)
    ws.fill_(0xFF)
    print(f"relaxed backward N={N} d={d} dpsi={dpsi} A={A}", flush=True)
    tr.router_relaxed_backward(c, B, T, x, psi, rw, p, fwd, eidx, egate, gin,
                               tr.RelaxGradOut(**{n: t.data_ptr() for n, t in out.items()}), ws)
    torch.cuda.synchronize()
    v = {n: t.double().requires_grad_(True) for n, t in dict(w, x=x, psi=psi).items()}
    n1 = v["x"] * torch.rsqrt(v["x"].square().mean(1, keepdim=True) + 1e-6) * v["g1"]
    a1 = torch.cat([n1, v["psi"]], 1) @ v["W1"].t() + v["b1"]
    h = (0.5 * a1 * (1 + torch.erf(a1 / 2 ** 0.5))) @ v["W2"].t() + v["b2"]
    hh = h * torch.rsqrt(h.square().mean(1, keepdim=True) + 1e-6) * v["gr"]
    za, ze, zb = (hh @ v[a].t() + v[b] for a, b in (("Wa", "ca"), ("We", "ce"), ("Wb", "cb")))
    za = za.view(N, A, 3)
    pe, sel = torch.softmax(ze, 1), eidx.long()
    gate = pe.gather(1, sel)
    gate = gate / gate.sum(1, keepdim=True)
    ya, yb = torch.softmax((za + ga) / 1.3, -1), torch.softmax((zb + gb) / 0.8, -1)
    loss = (up["a"] * ya).sum() / rho[0] + (up["e"] * gate).sum() / rho[1] + (up["b"] * yb).sum() / rho[2]
    st, us = o["stats"], o["usage_exp"]
    for z, f in ((za.reshape(-1, 3), st[tr.RS_F_ATTN:tr.RS_F_ATTN + 3]), (ze, us[0]),
                 (zb, st[tr.RS_F_BITS:tr.RS_F_BITS + 4])):
        P = torch.softmax(z, 1).mean(0)
        ent = -(P * P.log()).sum()
        loss = loss + 0.01 * len(f) * (f * P).sum() + 0.001 * torch.logsumexp(z, 1).square().mean() \
            + 0.1 * (0.99 * np.log(len(f)) - ent).clamp_min(0)
    loss.backward()
    for n, t in out.items():
        if t.numel():
            assert_close(npy(t), npy(v[n[1:]].grad), "f32", n)


def test_relaxed_backward_partial_sums():
    """120000 equal tokens: a head's weight gradient is the outer product of
    its bias gradient (their sum of dz, added in fp64) and the mean of h^.  Equal
    terms round alike, so the fp32 partial sums show their length: of n terms p
    the k-th addition errs by half an ulp of k p at most, 2^-24 k p, together
    2^-24 n / 2 of the sum; n is 128 tokens.  (fp64 adds the partial sums.)"""
    N, H, E, k, d, A, dev = 120000, 4, 3, 2, 64, 4, dict(device=DEV)
    c = tr.make_cfg(d, H, 2, 64, 64, E, k, 128, 64, "f32", attn_groups=0)
    g = torch.Generator(**dev)
    g.manual_seed(73)

    def rnd(*shape, std=1.0):
        return torch.randn(shape, generator=g, **dev) * std

    def same(*shape):
        return rnd(1, *shape).expand(N, *shape).contiguous()

    w = dict(g1=1 + rnd(d, std=0.02), W1=rnd(128, d + 8, std=0.05), b1=rnd(128, std=0.02),
             W2=rnd(128, 128, std=0.1), b2=rnd(128, std=0.02), gr=1 + rnd(128, std=0.02),
             Wa=rnd(3 * A, 128, std=0.1), ca=rnd(3 * A, std=0.1), We=rnd(E + 1, 128, std=0.1),
             ce=rnd(E + 1, std=0.1), Wb=rnd(4, 128, std=0.1), cb=rnd(4, std=0.1))
    rw = tr.RouterW(*(t.data_ptr() for t in w.values()))
    x, psi, ga, gb = same(d), same(8), same(A, 3), same(4)
    pos = torch.zeros(N, dtype=torch.int32, **dev)
    p = tr.RelaxParams(g_attn=ga.data_ptr(), g_bits=gb.data_ptr(), pos=pos.data_ptr(), tau_a=1.3,
                       tau_b=0.8)
    f64 = dict(dtype=torch.float64, **dev)
    o = dict(y_attn=torch.empty(N, A, 3, **dev), y_bits=torch.empty(N, 4, **dev),
             c_flops=torch.empty(N, **dev), c_mem=torch.empty(N, **dev),
             stats=torch.empty(tr.RELAX_NSTAT, **f64), usage_exp=torch.empty(2, E + 1, **f64),
             h_mean=torch.empty(128, **dev), h_var=torch.empty(128, **dev))
    fwd = tr.RelaxOut(**{n: v.data_ptr() for n, v in o.items()})
    eidx, egate = torch.empty(N, k, dtype=torch.int32, **dev), torch.empty(N, k, **dev)
    print(f"partial sums N={N}", flush=True)
    tr.router_relaxed(c, 1, N, x, psi, rw, p, torch.empty_like(x),
                      torch.empty(N, H, dtype=torch.uint8, **dev),
                      torch.empty(N, dtype=torch.uint8, **dev), eidx, egate,
                      tr.CompactionBuffers(c, 1, N).struct, fwd,
                      tr.workspace(c, tr.OP_ROUTER_RELAXED, 1, N))
    ua, ub, ue = same(A, 3), same(4), same(k)
    gin = tr.RelaxGradIn(g_attn=ua.data_ptr(), g_bits=ub.data_ptr(), g_gate=ue.data_ptr(), rho_m=0.0)
    out = {"d" + n: torch.empty_like(v) for n, v in w.items()}
    out.update(dx=torch.empty(N, d, **dev), dpsi=torch.empty(N, 8, **dev))
    tr.router_relaxed_backward(c, 1, N, x, psi, rw, p, fwd, eidx, egate, gin,
                               tr.RelaxGradOut(**{n: v.data_ptr() for n, v in out.items()}),
                               tr.workspace(c, tr.OP_ROUTER_RELAXED_BACKWARD, 1, N))
    torch.cuda.synchronize()
    h = npy(o["h_mean"]).astype(np.float64)
    for n in "aeb":
        ref = np.outer(npy(out["dc" + n]).astype(np.float64), h)
        on = np.abs(ref) > 0                     # (options outside the top k: zeros)
        assert on.mean() >= k / (E + 1) and not npy(out["dW" + n])[~on].any(), n
        err = np.abs(npy(out["dW" + n])[on] / ref[on] - 1).max() / 2.0 ** -24
        # the bias gradient, the mean and the result are each rounded once more
        note(f"dW{n} (bound 67 units of 2^-24)", err / 67)
        assert err <= 67, (n, err)


# ------------------------------------------- lists and slots beside other work
@pytest.mark.parametrize("B,T,prefill", [
    (1, 1, False), (512, 1, False), (513, 1, False),   # decode: one chunk of 1024 assignments, two
    (1, 1, True), (512, 1, True), (700, 1, True),      # prefill of single tokens, likewise
    (3, 171, True), (2, 1030, True),                   # slots ahead of the codes, 1 and 2 rounds
])
def test_layer_lists_and_slots(monkeypatch, B, T, prefill):
    """A layer's lists, slots and zeroed rows, made beside other kernels,
    against the stage calls on the layer's own decisions: the same lists feed
    the same kernels, so the results are the same bits; attention (split in
    the layer's prefill) at the tolerance of its bf16 output."""
    L = _small_layer(monkeypatch, B=B, T=T, H=4, Hkv=2, dh=64, w=100)
    D = DeviceLayer(L)
    c, N = D.cfg, B * T
    caches = [tr.KVCache(c, B, T + 40) for _ in range(2)]
    sid = torch.arange(B, dtype=torch.int32, device=DEV)
    sid[1:][-1:] = B                             # the last of several rows is outside the cache
    u8 = dict(dtype=torch.uint8, device=DEV)

    def act(*shape):
        return torch.full(shape, float("nan"), dtype=D.act, device=DEV)

    t = dict(q=act(N, 256), k=act(N, 128), v=act(N, 128), o=act(N, 256), xt=act(N, 256),
             mode=torch.empty(N, 4, **u8), bit=torch.empty(N, **u8),
             eidx=torch.empty(N, 2, dtype=torch.int32, device=DEV),
             egate=torch.empty(N, 2, device=DEV))
    x_out = act(N, 256)
    args = (B, T) if prefill else (B,)
    run, op = (tr.layer_prefill, tr.OP_LAYER_PREFILL) if prefill else \
        (tr.layer_decode, tr.OP_LAYER_DECODE)
    ws = tr.workspace(c, op, B, T)
    ws.fill_(0xFF)
    print(f"lists B={B} T={T} prefill={prefill}", flush=True)
    run(c, *args, D.x, D.psi, D.rw, D.dw, D.mw, caches[0], x_out, ws,
        taps=tr.Taps(**{n: v.data_ptr() for n, v in t.items()}), seq_ids=sid)
    cmp = tr.CompactionBuffers(c, B, T)
    mode, bit, eidx = (torch.empty_like(t[n]) for n in ("mode", "bit", "eidx"))
    tr.router(c, B, T, D.x, D.psi, D.rw, act(N, 256), mode, bit, eidx,
              torch.empty(N, 2, device=DEV), cmp.struct, tr.workspace(c, tr.OP_ROUTER, B, T))
    tr.kv_append(c, caches[1], B, T, t["k"], t["v"], bit, tr.workspace(c, tr.OP_KV_APPEND, B, T),
                 seq_ids=sid)
    o, y = act(N, 256), act(N, 256)
    if prefill:
        tr.attn_prefill(c, B, T, t["q"], caches[1], mode, cmp.struct, o, seq_ids=sid)
    else:
        tr.attn_decode(c, B, t["q"], caches[1], mode, o,
                       ws=tr.workspace(c, tr.OP_ATTN_DECODE, B, 1), seq_ids=sid)
    tr.moe(c, N, t["xt"], D.dw, D.mw, eidx, t["egate"], cmp.struct, y,
           tr.workspace(c, tr.OP_MOE, B, T))
    torch.cuda.synchronize()
    for n, v in (("mode", mode), ("bit", bit), ("eidx", eidx)):
        assert torch.equal(t[n], v), n
    assert torch.equal(x_out, y)
    assert torch.equal(caches[0].seq_len(), caches[1].seq_len())
    assert torch.equal(caches[0].pool_len(), caches[1].pool_len())
    assert caches[0].status() == caches[1].status() == (tr.CACHE_BAD_SEQ if B > 1 else 0)
    assert_close(npy(t["o"]), npy(o), "bf16", "o")
    zero = (t["mode"] == 0)
    if B > 1:
        zero[-T:] = True
    assert not t["o"].view(N, 4, 64)[zero].any()


# --------------------------------------------------------- controller's tail
@pytest.mark.parametrize("N,d,H,E,k,groups", [
    (1, 128, 2, 1, 1, 0), (256, 128, 4, 4, 1, 2),      # the form for few tokens
    (3, 3136, 16, 16, 2, 0),                           # its chunks are too many: tiles of one
    (257, 1024, 16, 16, 2, 0), (1000, 128, 4, 63, 5, 0),  # 2 and 4; 69 logits; 64 options
    (2048, 128, 30, 12, 13, 0), (2049, 128, 12, 8, 2, 1),  # 8, 107 logits, all taken; 16
    (8192, 128, 12, 8, 2, 0), (8193, 128, 12, 8, 2, 0),    # a tile a block; a block with two
    (24600, 128, 32, 4, 2, 16),                        # four tiles a block, heads past 16
])
def test_router_tail_tiles(N, d, H, E, k, groups):
    """The logits on both sides of the tail's tile rule against fp64, within
    the fp32 bound, and the decisions against the call's own logits: first
    maximum on ties (planted), gates within the rounding of k + 2 terms."""
    A, dev = groups or H, dict(device=DEV)
    c = tr.make_cfg(d, H, H // 2, 64, 64, E, k, 128, 64, "f32", d_psi=8, attn_groups=groups)
    g = torch.Generator(**dev)
    g.manual_seed(81)

    def rnd(*shape, std=1.0):
        return torch.randn(shape, generator=g, **dev) * std

    w = dict(g1=1 + rnd(d, std=0.02), W1=rnd(128, d + 8, std=0.6 * d ** -0.5), b1=rnd(128, std=0.02),
             W2=rnd(128, 128, std=0.1), b2=rnd(128, std=0.02), gr=1 + rnd(128, std=0.02),
             Wa=rnd(3 * A, 128, std=0.1), ca=rnd(3 * A, std=0.1), We=rnd(E + 1, 128, std=0.1),
             ce=rnd(E + 1, std=0.1), Wb=rnd(4, 128, std=0.1), cb=rnd(4, std=0.1))
    for m, b, i, j in (("Wa", "ca", 0, 2), ("We", "ce", 0, E), ("Wb", "cb", 1, 3)):  # equal logits
        w[m][j], w[b][j] = w[m][i].clone(), w[b][i].clone()
    rw = tr.RouterW(*(t.data_ptr() for t in w.values()))
    x, psi = rnd(N, d), rnd(N, 8)
    pos = torch.arange(N, dtype=torch.int32, **dev)
    ga, gb = rnd(N, A, 3), rnd(N, 4)
    p = tr.RelaxParams(g_attn=ga.data_ptr(), g_bits=gb.data_ptr(), pos=pos.data_ptr(), tau_a=1.3,
                       tau_b=0.8, zeta=0.99, alpha=0.01, beta=0.001, gamma=0.1)
    f64 = dict(dtype=torch.float64, **dev)
    z = torch.full((N, 3 * A + E + 5), float("nan"), **dev)
    o = dict(y_attn=torch.empty(N, A, 3, **dev), y_bits=torch.empty(N, 4, **dev),
             c_flops=torch.empty(N, **dev), c_mem=torch.empty(N, **dev), z=z,
             stats=torch.empty(tr.RELAX_NSTAT, **f64), usage_exp=torch.empty(2, E + 1, **f64))
    u8 = dict(dtype=torch.uint8, **dev)
    cmp = tr.CompactionBuffers(c, 1, N)
    mode, bit = torch.full((N, H), 9, **u8), torch.full((N,), 9, **u8)
    eidx, egate = torch.full((N, k), -1, dtype=torch.int32, **dev), torch.empty(N, k, **dev)
    print(f"router tail N={N} d={d} H={H} E={E} k={k}", flush=True)
    tr.router_relaxed(c, 1, N, x, psi, rw, p, torch.empty_like(x), torch.empty_like(mode),
                      torch.empty_like(bit), torch.empty_like(eidx), torch.empty_like(egate),
                      cmp.struct, tr.RelaxOut(**{n: t.data_ptr() for n, t in o.items()}),
                      tr.workspace(c, tr.OP_ROUTER_RELAXED, 1, N))
    ws = tr.workspace(c, tr.OP_ROUTER, 1, N)
    ws.fill_(0xFF)
    tr.router(c, 1, N, x, psi, rw, torch.empty_like(x), mode, bit, eidx, egate, cmp.struct, ws)
    torch.cuda.synchronize()
    v = {n: t.double() for n, t in dict(w, x=x, psi=psi).items()}
    n1 = v["x"] * torch.rsqrt(v["x"].square().mean(1, keepdim=True) + 1e-6) * v["g1"]
    a1 = torch.cat([n1, v["psi"]], 1) @ v["W1"].t() + v["b1"]
    h = (0.5 * a1 * (1 + torch.erf(a1 / 2 ** 0.5))) @ v["W2"].t() + v["b2"]
    h = h * torch.rsqrt(h.square().mean(1, keepdim=True) + 1e-6) * v["gr"]
    ref = torch.cat([h @ v["W" + n].t() + v["c" + n] for n in "aeb"], 1)
    assert_close(npy(z), npy(ref), "f32", "z")
    za, ze, zb = npy(z)[:, :3 * A].reshape(N, A, 3), npy(z)[:, 3 * A:-4], npy(z)[:, -4:]
    assert (npy(mode) == np.repeat(za.argmax(2), H // A, 1)).all()    # argmax: the first maximum
    assert (npy(bit) == zb.argmax(1)).all()
    sel = np.sort(np.argsort(-ze, 1, kind="stable")[:, :k], 1)
    assert (npy(eidx) == sel).all()
    e = np.exp(np.take_along_axis(ze, sel, 1).astype(np.float64) - ze.max(1, keepdims=True))
    gate = e / e.sum(1, keepdims=True)
    # exp to 2 ulp and the rounded difference it takes (|z| < 8: 2^-21), k + 1 sums, a division
    assert np.abs(npy(egate) / gate - 1).max() <= 2 * 2.0 ** -21 + (k + 6) * 2.0 ** -24


# ------------------------------------------------------- the append's quantizer
@pytest.mark.parametrize("dh,G,act", [(64, 32, "f32"), (128, 64, "f32"), (128, 32, "bf16")])
def test_append_codes_at_the_edges(dh, G, act):
    """Codes of groups where the quotient sits on or next to halfway points,
    where the fp16 scale is 0, subnormal or infinite, and where the fp16 zero
    is infinite (but no NaN arises): the same bytes as the oracle's division."""
    c, T, Hkv = tr.make_cfg(256, 2, 1, dh, 64, 4, 1, 128, G, act), 96, 1
    rng = gen.stream(91, "edges", dh, G)
    x = np.empty((2, T, Hkv, dh // G, G), np.float32)
    for i in range(2):
        for t in range(T):
            bits = (2, 4, 8)[t % 3]
            lv, u = 2 ** bits - 1, rng.random((Hkv, dh // G, G))
            scale = np.float16(2.0 ** rng.integers(-24, 10) * (1 + rng.integers(0, 1024) / 1024))
            kind = t // 3 % 8
            half = (rng.integers(0, lv, u.shape) + 0.5) * np.float64(scale)
            g = half * (1 + rng.choice([0, 6e-8, -6e-8, 2e-7, -2e-7], u.shape))
            g[..., 0], g[..., 1] = 0, lv * np.float64(scale)
            if kind == 1:
                g = g + np.float64(scale) * rng.integers(-8, 8)   # zero not 0
            elif kind == 2:
                g = np.full(u.shape, 0.3)                         # scale 0
            elif kind == 3:
                g = u * lv * 1.5e-7                               # subnormal scale
            elif kind == 4:
                g = u * 1e-9                                      # scale rounds to 0
            elif kind == 5:
                g = u * 3e37                                      # infinite scale
                g[..., 0] = 0
            elif kind == 6:
                g = u * lv - 1e5                                  # zero -inf
            elif kind == 7:
                g = u * lv + 1e5                                  # zero +inf
            x[i, t] = g
    x = gen.to_act(x.reshape(2, T, Hkv, dh), act)
    bit = (np.arange(T) % 3).astype(np.uint8)
    cache = tr.KVCache(c, 1, 128)
    _append(c, cache, 0, x[0], x[1], bit, act)
    for bi, nb in enumerate((2, 4, 8)):
        n = int((bit == bi).sum())
        ko = torch.zeros(n, Hkv, dh, dtype=torch.uint8, device=DEV)
        vo = torch.zeros_like(ko)
        ks = torch.zeros(n, Hkv, dh // G, 2, dtype=torch.int16, device=DEV)
        vs = torch.zeros_like(ks)
        tr.kv_export(c, cache, 0, bi, 0, n, ko, vo, ks, vs,
                     torch.zeros(n, dtype=torch.int32, device=DEV))
        torch.cuda.synchronize()
        for src, out, sz in ((x[0], ko, ks), (x[1], vo, vs)):
            with np.errstate(over="ignore"):
                codes, s16, z16 = oracle.quant.quantize(src[bit == bi], nb, G)
            np.testing.assert_array_equal(npy(out), codes)
            np.testing.assert_array_equal(npy(sz)[..., 0], s16.view(np.int16))
            np.testing.assert_array_equal(npy(sz)[..., 1], z16.view(np.int16))
