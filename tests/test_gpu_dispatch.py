"""Edges of the size rules that choose between kernels and launch shapes, each
against the CPU oracle (through the C ABI) at the repository's tolerances."""
import numpy as np
import pytest
import torch

import gen
import oracle
import paper_2607_06601_amd as tr
from paper_2607_06601_amd.device import to_dev

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
