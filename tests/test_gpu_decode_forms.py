"""Decode attention in every form of its kernels (keys and values in one
wavefront or in two, up to 4 and up to 8 query heads per KV head, one table or
two, compiled and general record lengths, fixed-width records, per-token streams
at p = 8 and 12, contiguous and paged): against 64 bits, closely enough that
every digit of the fixed-point operands counts, with scales of both signs and
zero; and at a sequence's end, where record rows past the length may hold
anything."""

from dataclasses import dataclass

import numpy as np
import pytest
import torch

import dq_workloads as wlmod
import paper_2609_19880_amd as dq
from oracle import attention, fixed, hadamard, kmean, kv, tables

DEV = "cuda:0"
B, LENS = 2, (1373, 130)         # last tiles of 29 and 2 live tokens


@dataclass(frozen=True)
class Form:
    name: str
    H: int
    G: int
    ck: tuple                    # (levels, record bytes, p) of the keys; None: fixed-width records
    cv: tuple
    cap: int                     # the chunk follows the capacity: a small one gives split tiles
    token: bool = False
    page: int = 0


SIX, FIVE, SEVENTEEN = (6, 36, 12), (5, 32, 12), (17, 64, 12)
FORMS = [
    Form("split", 2, 4, SIX, SIX, 1408),
    Form("whole", 2, 4, SIX, SIX, 131072),
    Form("g3", 2, 3, FIVE, FIVE, 131072),
    Form("g8", 2, 8, SIX, SIX, 1408),
    Form("g6_two_tables", 2, 6, (9, 48, 12), FIVE, 131072),
    Form("two_tables", 2, 4, (6, 36, 10), FIVE, 1408),
    Form("general_lengths", 2, 4, (6, 40, 12), (6, 36, 12), 1408),
    Form("paged", 2, 4, SIX, SIX, 2048, page=256),
    Form("fixed", 2, 4, None, None, 1408),
    Form("token_split", 2, 4, (8, 88, 8), (6, 62, 8), 1408, token=True),
    Form("token_whole", 2, 4, (8, 88, 8), (6, 62, 8), 131072, token=True),
    Form("token_whole_p12", 2, 3, (8, 88, 12), (6, 62, 12), 131072, token=True),
    Form("token_g8", 2, 8, (8, 88, 8), (6, 62, 8), 131072, token=True),
    Form("token_paged", 2, 4, (8, 88, 8), (6, 62, 8), 2048, token=True, page=256),
]


class Cache:
    """Keys (with means) and values coded by the library into buffers of the
    form's layout."""

    def __init__(self, f: Form, seed: int):
        self.f = f
        rng = np.random.default_rng(seed)
        T = (max(LENS) + 127) // 128 * 128
        wl = wlmod.workload("b1_t4k")
        w = wlmod.Workload("forms", B, T, f.H * f.G, f.H, 4, wl.k, wl.v)
        k, v, self.q = wlmod.make_k(w, seed).to(DEV), wlmod.make_v(w, seed).to(DEV), wlmod.make_q(w, seed).to(DEV)
        self.status = torch.zeros(1, dtype=torch.int32, device=DEV)
        self.lens = torch.tensor(LENS, dtype=torch.int32, device=DEV)
        self.ws = torch.empty(dq.dq_decode_workspace_bytes(B, f.H * f.G, f.H, f.cap), dtype=torch.uint8, device=DEV)
        cap, n = f.cap, 128 * f.H if f.token else 128
        u8, i8, i16 = torch.uint8, torch.int8, torch.int16
        self.bt = None
        if f.ck is None:
            self.C = (36, 36)
        else:
            self.C = (f.ck[1], f.cv[1])
            self.tk = dq.Tables(n, f.ck[0], f.ck[2], f.ck[1], 1.4)
            self.tv = self.tk if f.ck == f.cv else dq.Tables(n, f.cv[0], f.cv[2], f.cv[1], 1.4)
        if f.page:
            pages = B * cap // f.page
            self.bt = torch.from_numpy(rng.permutation(pages).astype(np.int32).reshape(B, -1)).to(DEV)
            lead = (pages, f.page)
        else:
            lead = (B, cap)
        if f.token and f.page:
            self.rec = [torch.zeros(dq.token_pool_shape(t, *lead), dtype=u8, device=DEV) for t in (self.tk, self.tv)]
        elif f.token:
            self.rec = [torch.zeros(dq.token_records_shape(t, *lead), dtype=u8, device=DEV) for t in (self.tk, self.tv)]
        else:
            self.rec = [torch.zeros((lead[0], f.H, lead[1], C), dtype=u8, device=DEV) for C in self.C]
        self.mq = torch.zeros((lead[0], f.H, lead[1] // 128, 128), dtype=i8, device=DEV)
        self.ms = torch.zeros((lead[0], f.H, lead[1] // 128), dtype=i16, device=DEV)
        for i, x in enumerate((k, v)):
            means = (self.mq, self.ms) if i == 0 else (None, None)
            if f.ck is None:
                dq.dq_encode_kv_fixed(128, 36, x, 0, cap, self.rec[i], *means, self.status)
                continue
            tab = (self.tk, self.tv)[i]
            if f.page:
                call = dq.dq_encode_kv_token_paged if f.token else dq.dq_encode_kv_paged
                call(tab, x, 0, self.bt, self.rec[i], *means, self.status)
            else:
                call = dq.dq_encode_kv_token if f.token else dq.dq_encode_kv
                call(tab, x, 0, cap, self.rec[i], *means, self.status)
        torch.cuda.synchronize()
        assert int(self.status.item()) == 0

    def rows(self, i, b):
        """Records of sequence b, a view per tile or page and KV head: yields
        (first token, [tokens, bytes] view that writes through)."""
        f, r = self.f, self.rec[i]
        if f.token:
            per = f.page // 64 if f.page else r.shape[1]
            for t in range(0, f.cap, 64):
                page, tile = (int(self.bt[b, t // f.page]), t // 64 % per) if f.page else (b, t // 64)
                yield t, r[page, tile].permute(1, 0, 2)           # [64, S / 8, 8]
                if t >= 2048:
                    return
        elif f.page:
            for j in range(f.cap // f.page):
                for h in range(f.H):
                    yield j * f.page, r[int(self.bt[b, j]), h]
        else:
            for h in range(f.H):
                yield 0, r[b, h, :2048]

    def levels(self, i, b):
        """Levels [H, T, 128], scales and offsets [H, T] of sequence b."""
        f, T = self.f, LENS[b]
        parts = sorted(((t, j, rows.cpu().numpy()) for j, (t, rows) in enumerate(self.rows(i, b)) if t < T),
                       key=lambda e: e[:2])
        n, per_head = (128 * f.H, 1) if f.token else (128, f.H)
        rec = np.concatenate([r.reshape(1, r.shape[0], -1) for _, _, r in parts])
        rec = rec.reshape(-1, per_head, *rec.shape[1:]).transpose(1, 0, 2, 3)
        rec = np.ascontiguousarray(rec.reshape(per_head, -1, rec.shape[-1])[:, :T, :self.C[i]])
        if f.ck is None:
            return fixed.unpack(rec, 128, 2)
        M, C, p = (f.ck, f.cv)[i]
        sym, s, o, ok = kv.decode_records(rec, tables.build_tables(n, M, p, 1.4, C), n)
        assert ok.all()
        return tuple(x[0] for x in kv.tokenwise_as_heads(sym, s, o, f.H)) if f.token else (sym, s, o)

    def means(self, b):
        """Dequantized key means [H, windows, 128]."""
        rows = self.bt[b].long() if self.f.page else [b]
        mq, ms = (x[rows].transpose(0, 1).flatten(1, 2).contiguous().cpu().numpy() for x in (self.mq, self.ms))
        return kmean.dequantize_mean(mq, ms.view(np.float16))[:, :(LENS[b] + 127) // 128]

    def fill_past_end(self, i, header, body):
        """Rows from the length on: the first four bytes (fp16 scale and
        offset) as given, the rest `body`."""
        for b, T in enumerate(LENS):
            for t, rows in self.rows(i, b):
                lo = max(0, T - t)
                if lo >= rows.shape[0]:
                    continue
                rows[lo:] = body
                for j, c in enumerate(header):
                    if rows.dim() == 3:
                        rows[lo:, 0, j] = c
                    else:
                        rows[lo:, j] = c

    def step(self, scale=None):
        f, out = self.f, torch.empty(self.q.shape, dtype=torch.float32, device=DEV)
        a = (self.lens, self.ws)
        kw = dict(softmax_scale=scale, status=self.status)
        if f.ck is None:
            dq.dq_decode_attention_fixed_partial(self.q, self.rec[0], self.mq, self.ms, self.rec[1], *a, **kw)
        elif f.page:
            call = dq.dq_decode_attention_token_paged_partial if f.token else dq.dq_decode_attention_paged_partial
            call(self.tk, self.tv, self.q, self.rec[0], self.mq, self.ms, self.rec[1], self.bt, *a, **kw)
        else:
            call = dq.dq_decode_attention_token_partial if f.token else dq.dq_decode_attention_partial
            call(self.tk, self.tv, self.q, self.rec[0], self.mq, self.ms, self.rec[1], *a, **kw)
        dq.dq_decode_attention_merge(B, f.H * f.G, f.H, self.lens, f.cap, self.ws, out)
        torch.cuda.synchronize()
        assert int(self.status.item()) == 0
        return out.cpu().numpy().astype(np.float64)


by_form = pytest.mark.parametrize("form", FORMS, ids=lambda f: f.name)


@pytest.mark.gpu
@by_form
def test_rows_past_the_length_are_ignored(form):
    """NaN or infinite scales and offsets, and any payload, in the rows that
    share the last tile with live tokens (a truncated sequence, a page used
    before): bit for bit the output over rows of zeros."""
    c = Cache(form, 61)
    for i in (0, 1):
        c.fill_past_end(i, (0, 0, 0, 0), 0)
    want = c.step()
    one, nan, inf, ninf = (0x00, 0x3C), (0x00, 0x7E), (0x00, 0x7C), (0x00, 0xFC)
    for s, o, body in ((nan, one, 0), (inf, one, 0x5A), (ninf, one, 0), (one, nan, 0), (one, inf, 0xFF), (nan, nan, 0xFF)):
        for i in (0, 1):
            c.fill_past_end(i, s + o, body)
        got = c.step()
        assert np.array_equal(got, want), (s, o, np.abs(got - want).max())


# Query and weights are 22-bit fixed point, sums and softmax fp32: 1e-6 to 3e-6
# from 64 bits (relative 2-norm over a sequence's heads).  Without the lowest of
# the three digits of either operand it would be 6e-5 and more.
LIMIT = 1.2e-5


def _without_digit(v, digit):
    """Integers v less their digit-th signed 8-bit digit."""
    if digit is None:
        return v
    w = (v.astype(np.int64) + 0x808080) ^ 0x808080
    return v - ((((w >> (8 * digit)) & 255) ^ 128) - 128) * 256.0 ** digit


def fixed_point(q, keys, mu, values, scale, query=None, weight=None):
    """One query head in the kernels' arithmetic: the rotated query in units of
    its largest value / 2^22, the weights (value scales folded in) in those of
    their 64-token tile's; the rest in 64 bits.  query, weight: the digit that
    is left out."""
    (ks, s, o), (vs, sv, ov) = keys, values
    qr, T = hadamard.fwht(q), len(s)
    unit = np.abs(qr).max() / 2 ** 22
    dot = ks @ (_without_digit(np.rint(qr / unit), query) * unit)
    logit = (s * dot + o * qr.sum() + np.repeat(mu @ qr, 128)[:T]) * scale / 128
    p = np.exp(logit - logit.max())
    acc = np.full(128, (p * ov).sum())
    for t in range(0, T, 64):
        w = p[t:t + 64] * sv[t:t + 64]
        unit = w.max() / 2 ** 22
        acc += (_without_digit(np.rint(w / unit), weight) * unit) @ vs[t:t + 64]
    return hadamard.fwht(acc) / 128 / p.sum()


def _error(got, want):
    return np.linalg.norm(got - want) / np.linalg.norm(want)


@pytest.mark.gpu
@by_form
@pytest.mark.parametrize("sign", [1, -1, 0])
def test_step_against_64_bits(form, sign):
    """Keys with non-zero means, lengths that end inside a tile; and, for the
    limit's worth, the same arithmetic less one digit does not meet it."""
    c = Cache(form, 62)
    assert bool((c.ms != 0).any())
    scale = sign / np.sqrt(128)
    got, q, G = c.step(float(scale)), c.q.cpu().double().numpy(), form.G
    for b, T in enumerate(LENS):
        keys, values = ([x.astype(np.float64) for x in c.levels(i, b)] for i in (0, 1))    # (levels, scales, offsets)
        mu = c.means(b)
        want = attention.attention_folded(q[b:b + 1], *(x[None] for x in keys), mu[None], *(x[None] for x in values),
                                          [T], G, scale)[0]
        assert _error(got[b], want) < LIMIT, b

        def model(**less):
            return np.stack([fixed_point(q[b, g], [x[g // G] for x in keys], mu[g // G], [x[g // G] for x in values],
                                         scale, **less) for g in range(form.H * G)])

        assert _error(model(), want) < LIMIT / 2
        # (at a scale of 0 the query has no part, and equal weights err alike)
        for digit in range(3 if sign else 0):
            assert _error(model(query=digit), want) > 3 * LIMIT
            assert _error(model(weight=digit), want) > 3 * LIMIT


@pytest.mark.gpu
@by_form
@pytest.mark.parametrize("size", [2e5, 1e10, 1e30])
def test_scores_of_any_size(form, size):
    """Queries so large that the scores' spacing exceeds an exponent's range: the
    softmax is one token's weight, and finite."""
    c = Cache(form, 63)
    c.q = (c.q.float() * size).to(torch.bfloat16)
    got, q, G = c.step(), c.q.cpu().double().numpy(), form.G
    for b, T in enumerate(LENS):
        keys, values = ([x.astype(np.float64) for x in c.levels(i, b)] for i in (0, 1))
        want = attention.attention_folded(q[b:b + 1], *(x[None] for x in keys), c.means(b)[None],
                                          *(x[None] for x in values), [T], G, 1 / np.sqrt(128))[0]
        assert np.isfinite(got[b]).all()
        assert _error(got[b], want) < LIMIT, b
