"""Edges of the size rules that choose between kernels and launch shapes, each
against the CPU oracle (through the C ABI) at the repository's tolerances."""
import numpy as np
import pytest
import torch

import gen
import oracle
import paper_2607_06601_amd as tr
from paper_2607_06601_amd.device import DeviceLayer, to_dev

from _common import assert_close, npy, torch_act

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
    (3, 33, 8, 1, 64, 300, 0, None),         # two quartets, chunks without a key
    (1, 400, 4, 4, 128, 256, 1100, None),    # one head per kv head
])
def test_prefill_split_key_ranges(monkeypatch, B, T, H, Hkv, dh, w, ctx, pages):
    """The layer's attention (key ranges split over its scratch) against the
    stage call (never split) on the same queries, modes and cache: both round
    the same sums, taken in another order, to bf16."""
    L = _small_layer(monkeypatch, B=B, T=T, H=H, Hkv=Hkv, dh=dh, w=w)
    D = DeviceLayer(L)
    c, N = D.cfg, B * T
    n_seq, cap = B + 2, 20000 if ctx else 4096   # chunk counts follow the capacity
    pg = None if pages is None else (pages, [64] * 4)
    cache = tr.KVCache(c, n_seq, cap, pages=pg)
    rng = gen.stream(41, "split", T, ctx)
    ids = list(rng.permutation(n_seq)[:B])
    if ctx:
        for s in ids:
            n = int(ctx * (0.5 + 0.5 * rng.random()))
            k, v = gen.kv_block(41 + int(s), n, Hkv, dh, "bf16", 0.8)
            _append(c, cache, int(s), k, v, rng.integers(0, 4, n).astype(np.uint8), "bf16")
    if B > 2:
        ids[1] = n_seq                           # a row outside the cache: zeros
    sid = torch.tensor([int(s) for s in ids], dtype=torch.int32, device=DEV)
    t = dict(q=torch.empty(N, H * dh, dtype=D.act, device=DEV),
             o=torch.full((N, H * dh), float("nan"), dtype=D.act, device=DEV),
             mode=torch.empty(N, H, dtype=torch.uint8, device=DEV))
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
