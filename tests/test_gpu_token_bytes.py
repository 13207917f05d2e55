"""Per-token decode attention over records that stress how it reads bytes at
each precision: streams of the rarest symbol (at p = 8 one byte in every step,
the most a step can read), of the commonest (no byte for many steps), both in
long runs, and random ones, at lengths around tile and chunk ends; in both forms
of the kernel (small chunks: keys and values in different wavefronts); and a
record whose state starts below its range, which has to be flagged."""

import numpy as np
import pytest
import torch

import dq_workloads as wlmod
import paper_2609_19880_amd as dq
from oracle import attention, kv, rans, tables
from tokrec import to_tiles

pytestmark = pytest.mark.gpu

DEV = "cuda:0"
TOL = 2e-3


def _records(rng, tab, n, count):
    f = tab.freq
    rare, common = int(np.argmin(f)), int(np.argmax(f))
    sym = np.empty((count, n), dtype=np.int64)
    for i in range(count):
        k = i % 5
        if k == 0:
            sym[i] = rare
        elif k == 1:
            sym[i] = common
        elif k == 2:
            sym[i] = np.where(np.arange(n) // 37 % 2, rare, common)
        elif k == 3:
            sym[i] = np.where(rng.random(n) < 0.5, rare, rng.integers(tab.M, size=n))
        else:
            sym[i] = rng.choice(tab.M, size=n, p=f / f.sum())
    s16 = rng.uniform(0.5, 2.0, size=count).astype(np.float16)
    o16 = rng.normal(size=count).astype(np.float16)
    state, body, length = rans.encode(sym, tab)
    assert int(np.max(length)) + 8 <= tab.record_bytes
    return rans.pack(s16, o16, state, body, length, tab.record_bytes), sym, s16, o16


@pytest.mark.parametrize("pk,pv", [(8, 8), (8, 12), (12, 8), (9, 9)])
@pytest.mark.parametrize("H,G,T,cap", [(8, 4, 193, 256), (8, 4, 193, 65536), (8, 8, 130, 256), (2, 3, 64, 128),
                                       (4, 1, 257, 65536), (1, 4, 1, 128)])
def test_token_attention_over_stressed_records(pk, pv, H, G, T, cap):
    n = 128 * H
    # room for every symbol at its dearest
    Ck, Cv = n * pk // 8 + 16, n * pv // 8 + 16
    gtk, gtv = dq.Tables(n, 8, pk, Ck, 1.4), dq.Tables(n, 6, pv, Cv, 1.4)
    otk, otv = tables.build_tables(n, 8, pk, 1.4, Ck), tables.build_tables(n, 6, pv, 1.4, Cv)
    rng = np.random.default_rng(n + pk * 100 + pv + T)
    tiles = (T + 127) // 128 * 128
    krec, ksym, ks, ko = _records(rng, otk, n, tiles)
    vrec, vsym, vs, vo = _records(rng, otv, n, tiles)
    Sk, Sv = dq.dq_token_record_stride(gtk), dq.dq_token_record_stride(gtv)
    gk = torch.zeros(dq.token_records_shape(gtk, 1, cap), dtype=torch.uint8, device=DEV)
    gv = torch.zeros(dq.token_records_shape(gtv, 1, cap), dtype=torch.uint8, device=DEV)
    gk[:, :tiles // 64] = torch.from_numpy(to_tiles(krec[None], Sk)).to(DEV)
    gv[:, :tiles // 64] = torch.from_numpy(to_tiles(vrec[None], Sv)).to(DEV)
    mq = torch.zeros((1, H, cap // 128, 128), dtype=torch.int8, device=DEV)
    ms = torch.zeros((1, H, cap // 128), dtype=torch.int16, device=DEV)
    q = torch.from_numpy(rng.normal(size=(1, H * G, 128)).astype(np.float32)).to(torch.bfloat16)
    lens = torch.tensor([T], dtype=torch.int32, device=DEV)
    ws = torch.empty(dq.dq_decode_workspace_bytes(1, H * G, H, cap), dtype=torch.uint8, device=DEV)
    status = torch.zeros(1, dtype=torch.int32, device=DEV)

    def step(scale):
        out = torch.empty((1, H * G, 128), dtype=torch.float32, device=DEV)
        dq.dq_decode_attention_token_partial(gtk, gtv, q.to(DEV), gk, mq, ms, gv, lens, ws, softmax_scale=scale,
                                             status=status)
        dq.dq_decode_attention_merge(1, H * G, H, lens, cap, ws, out)
        return out.cpu().numpy().astype(np.float64)

    kh = kv.tokenwise_as_heads(ksym[None], ks[None], ko[None], H)
    vh = kv.tokenwise_as_heads(vsym[None], vs[None], vo[None], H)
    qd = kv.bf16_to_f64(wlmod.bf16_bits(q))
    # a softmax scale of either sign, and none at all
    for scale in (1 / np.sqrt(128), -0.05, 0.0):
        ref = attention.attention_folded(qd, *kh, None, *vh, [T], G, scale)
        got = step(scale)
        err = np.max(np.abs(got - ref) / np.max(np.abs(ref), axis=-1, keepdims=True))
        assert err < TOL, (scale, err)
    assert int(status.item()) == 0
    # a state below the range, key or value, in the last live token
    for buf, S in ((gk, Sk), (gv, Sv)):
        t = T - 1
        row = buf[0, t // 64, 0, t % 64]
        keep = row.clone()
        row[4:8] = torch.tensor([1, 0, 0, 0], dtype=torch.uint8, device=DEV)
        status.zero_()
        assert np.isfinite(step(1 / np.sqrt(128))).all()
        assert int(status.item()) & dq.DQ_STATUS_CORRUPT
        row.copy_(keep)
