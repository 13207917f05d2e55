"""The encoder's threshold search against the oracle where it can go wrong:
every way rates decide its form (two to four thresholds in registers, any
number, the outermost pair sharing their mean, rates it does not take), stream
lengths, record sizes that are no multiple of 4, and streams it must hand back
to the plain search (values on a tie, a few distinct values, a large offset).
These are small appends, of 4 streams per workgroup; those of 8 to 64 (32 per
token), with partly filled last workgroups, are compared with them."""

import numpy as np
import pytest
import torch

import dq_workloads as wlmod
import paper_2609_19880_amd as dq
from oracle import kv, tables
from tokrec import from_tiles

pytestmark = pytest.mark.gpu

DEV = "cuda:0"


def _streams(seed, B, T, H, d):
    """Values [B, T, H, d] bf16: token t follows pattern t mod 6."""
    rng = np.random.default_rng(seed)
    v = rng.normal(size=(B, T, H, d)).astype(np.float32)
    k = np.arange(T) % 6
    v[:, k == 1] = np.rint(v[:, k == 1] * 2)                       # small integers
    v[:, k == 2] = rng.choice([-1.0, 0.0, 1.0], size=v[:, k == 2].shape)
    v[:, k == 3, :, 0] += 300.0                                    # an offset far above the spread
    v[:, k == 4] *= rng.lognormal(0.0, 2.0, size=v[:, k == 4].shape[:2])[:, :, None, None]
    v[:, k == 5] = rng.laplace(size=v[:, k == 5].shape)            # heavy tails
    return torch.from_numpy(v).to(torch.bfloat16)


# (levels, record bytes, alpha, precision): the form the rates select
CODINGS = [(3, 30, 1.4, 12), (4, 34, 1.4, 10), (5, 32, 1.4, 12), (6, 37, 1.4, 12), (7, 42, 1.4, 9), (8, 43, 1.4, 12),
           (9, 48, 1.4, 12), (10, 50, 1.4, 12), (17, 64, 1.4, 12), (16, 36, 5.6, 12), (32, 48, 7.6, 12), (2, 26, 1.4, 8)]


@pytest.mark.parametrize("levels,C,alpha,p", CODINGS)
@pytest.mark.parametrize("prerotated", [False, True])
def test_search_matches_oracle_per_head(levels, C, alpha, p, prerotated):
    B, T, H = 1, 203, 2
    tab = dq.Tables(128, levels, p, C, alpha, prerotated)
    ot = tables.build_tables(128, levels, p, alpha, C)
    x = _streams(levels * 100 + C, B, T, H, 128)
    rec = torch.zeros((B, H, 256, C), dtype=torch.uint8, device=DEV)
    status = torch.zeros(1, dtype=torch.int32, device=DEV)
    dq.dq_encode_kv(tab, x.to(DEV), 0, 256, rec, None, None, status)
    want, _ = kv.encode_values(wlmod.bf16_bits(x), ot, rotate_on=not prerotated)
    got = rec.cpu().numpy()[:, :, :T]
    bad = np.argwhere((got != want).any(axis=-1))
    assert len(bad) == 0, f"{len(bad)} records differ, first {bad[:3].tolist()}"
    assert not rec[:, :, T:].any()


@pytest.mark.parametrize("d,levels,C", [(64, 6, 22), (64, 8, 26), (256, 6, 70), (256, 9, 90), (256, 17, 130)])
def test_search_matches_oracle_head_dims(d, levels, C):
    B, T, H = 1, 70, 1
    alpha = dq.smallest_feasible_alpha(d, levels, 12, C)
    tab = dq.Tables(d, levels, 12, C, alpha)
    ot = tables.build_tables(d, levels, 12, alpha, C)
    x = _streams(d + levels, B, T, H, d)
    rec = torch.zeros((B, H, 128, C), dtype=torch.uint8, device=DEV)
    dq.dq_encode_kv(tab, x.to(DEV), 0, 128, rec)
    want, _ = kv.encode_values(wlmod.bf16_bits(x), ot)
    assert np.array_equal(rec.cpu().numpy()[:, :, :T], want)


@pytest.mark.parametrize("H,levels,C,p", [(8, 8, 335, 8), (8, 6, 235, 8), (8, 8, 331, 12), (8, 17, 460, 12),
                                          (4, 8, 169, 8), (4, 6, 119, 8), (2, 9, 96, 12), (1, 6, 36, 12)])
def test_search_matches_oracle_per_token(H, levels, C, p):
    B, T = 2, 77
    alpha = dq.smallest_feasible_alpha(128 * H, levels, p, C)
    tab = dq.Tables(128 * H, levels, p, C, alpha)
    ot = tables.build_tables(128 * H, levels, p, alpha, C)
    x = _streams(H * 10 + levels, B, T, H, 128)
    rec = torch.zeros(dq.token_records_shape(tab, B, 128), dtype=torch.uint8, device=DEV)
    dq.dq_encode_kv_token(tab, x.to(DEV), 0, 128, rec)
    got = from_tiles(rec.cpu().numpy())[:, :T, :C]
    want = kv.encode_values_tokenwise(wlmod.bf16_bits(x), ot)[0]
    assert np.array_equal(got, want)


def _streams_per_group(most, tokens, rows):
    """The grid's rule: as many streams per workgroup as leave four workgroups per CU."""
    ns, cus = most, torch.cuda.get_device_properties(0).multi_processor_count
    while ns > 4 and -(-tokens // ns) * rows < 4 * cus:
        ns //= 2
    return ns


def _batch(seed, B, T, H):
    """[B, T, H, 128]: eight sequences, then the same with their channels rotated."""
    x = _streams(seed, min(B, 8), T, H, 128).to(DEV)
    return torch.stack([torch.roll(x[b % 8], b // 8, dims=-1) for b in range(B)])


# (sequences, streams per workgroup): 203 tokens leave 11 or 3 for the last one
@pytest.mark.parametrize("levels,C,alpha", [(6, 36, 1.4), (9, 47, 1.4), (32, 48, 7.6)])
@pytest.mark.parametrize("B,ns", [(5, 8), (10, 16), (20, 32), (32, 64)])
def test_records_do_not_depend_on_the_grid_per_head(B, ns, levels, C, alpha):
    """A batch in one append against its sequences one at a time."""
    T, H = 203, 8
    assert _streams_per_group(64, T, H * B) == ns and _streams_per_group(64, T, H) == 4
    tab = dq.Tables(128, levels, 12, C, alpha)
    x = _batch(B, B, T, H)
    whole, parts = (torch.zeros((B, H, 256, C), dtype=torch.uint8, device=DEV) for _ in range(2))
    dq.dq_encode_kv(tab, x, 0, 256, whole)
    for b in range(B):
        dq.dq_encode_kv(tab, x[b:b + 1], 0, 256, parts[b:b + 1])
    assert torch.equal(whole, parts)
    assert not whole[:, :, T:].any()


@pytest.mark.parametrize("levels,C,p", [(8, 335, 8), (17, 460, 12)])
@pytest.mark.parametrize("B,ns", [(40, 8), (79, 16), (147, 32)])
def test_records_do_not_depend_on_the_grid_per_token(B, ns, levels, C, p):
    """Symbols packed (8 levels) and not (17)."""
    T, H = 203, 8
    assert _streams_per_group(32, T, B) == ns and _streams_per_group(32, T, 1) == 4
    tab = dq.Tables(128 * H, levels, p, C, 1.4)
    x = _batch(B, B, T, H)
    whole, parts = (torch.zeros(dq.token_records_shape(tab, B, 256), dtype=torch.uint8, device=DEV) for _ in range(2))
    dq.dq_encode_kv_token(tab, x, 0, 256, whole)
    for b in range(B):
        dq.dq_encode_kv_token(tab, x[b:b + 1], 0, 256, parts[b:b + 1])
    assert torch.equal(whole, parts)


@pytest.mark.parametrize("B,T,whole_ns,part_ns", [(5, 384, 8, 4), (10, 384, 16, 8), (20, 384, 32, 16), (16, 1024, 64, 16)])
def test_caches_do_not_depend_on_the_grid(B, T, whole_ns, part_ns):
    """Keys with means and values: the same bytes as the same tokens appended
    one window at a time."""
    H = 8
    assert (_streams_per_group(64, T, H * B), _streams_per_group(64, 128, H * B)) == (whole_ns, part_ns)
    tab = dq.Tables(128, 6, 12, 36, 1.4)
    x = _batch(B + T, B, T, H)
    whole = dq.KVCache(B, H, H, T, tab, tab, device=DEV)
    parts = dq.KVCache(B, H, H, T, tab, tab, device=DEV)
    whole.append(x, x, 0)
    for t in range(0, T, 128):
        parts.append(x[:, t:t + 128], x[:, t:t + 128], t)
    for name in ("k_records", "v_records", "k_mean_q", "k_mean_scale", "status"):
        assert torch.equal(getattr(whole, name), getattr(parts, name)), name


@pytest.mark.parametrize("d,H,levels,C", [(64, 1, 6, 22), (128, 2, 2, 26), (128, 2, 6, 36), (256, 1, 9, 90)])
def test_zeros_of_both_signs(d, H, levels, C):
    """Streams of zeros that come rotated already: scale 0, and as the offset a
    zero whose sign is the smallest's where the reduction over the wavefront
    ends, channels 4, 68, ...: the bytes do not change with the layout of the
    channels over the lanes."""
    T = 96
    alpha = dq.smallest_feasible_alpha(d, levels, 12, C)
    tab = dq.Tables(d, levels, 12, C, alpha, True)
    neg = torch.from_numpy(np.random.default_rng(d + levels).random((1, T, H, d)) < 0.3)
    x = torch.where(neg, -0.0, 0.0).to(torch.bfloat16)
    rec = torch.zeros((1, H, 128, C), dtype=torch.uint8, device=DEV)
    dq.dq_encode_kv(tab, x.to(DEV), 0, 128, rec)
    head = rec[0, :, :T, :4].cpu()
    want = neg[0, :, :, 4::64].any(dim=-1).T
    assert bool(want.any()) and not bool(want.all())
    assert not head[:, :, :3].any() and torch.equal(head[:, :, 3], want.to(torch.uint8) * 0x80)
