"""Wavefronts per workgroup that the LDS layouts of the decode kernels leave
(CPU only: needs hipcc).  A wavefront's region holds what its two streams need
while they are decoded (byte pairs, or the two rings) and the tiles of its
products, nothing else: what is added to it costs wavefronts at the large
tables, where no timed call looks."""

import os
import shutil
import subprocess

import pytest

LDS, ROW = 160 * 1024, 80
# (p keys, p values, one table, record bytes, query heads per KV head, wavefronts)
HEAD = [
    (12, 12, True, 36, 36, 4, 16), (12, 12, True, 32, 32, 4, 16), (12, 12, True, 48, 48, 8, 8),
    (12, 10, False, 32, 32, 4, 16), (12, 11, False, 32, 32, 1, 16), (8, 11, False, 32, 32, 4, 16),
    (12, 12, False, 48, 32, 8, 8), (12, 12, False, 64, 64, 4, 4),
]
# (p keys, p values, one table, KV heads, query heads per KV head, chunk, wavefronts)
TOKEN = [
    (8, 8, False, 8, 4, 2048, 12), (12, 12, True, 8, 4, 2048, 10), (11, 11, False, 8, 4, 2048, 10),
    (12, 12, False, 8, 7, 2048, 5), (12, 12, False, 8, 8, 2048, 5), (11, 11, False, 8, 8, 512, 8),
    (8, 8, False, 8, 8, 2048, 8), (12, 12, False, 4, 1, 1024, 8),
]


def _syntax_check(tmp_path, source, asserts):
    import __graft_entry__ as ge

    if not os.path.exists(ge.HIPCC) and shutil.which("hipcc") is None:
        pytest.skip("hipcc not available")
    cpp = tmp_path / "layout.hip"
    cpp.write_text(f'#include "{os.path.join(ge.CSRC, source)}"\nnamespace dq {{\n' + "\n".join(asserts) + "\n}\n")
    flags = [f for f in ge.FLAGS if f not in ("-shared", "-fPIC")]
    res = subprocess.run([ge.HIPCC, *flags, "--cuda-host-only", "-fsyntax-only", str(cpp)], capture_output=True,
                         text=True)
    assert res.returncode == 0, res.stderr[-3000:]


def test_per_head_wavefronts(tmp_path):
    asserts = []
    for pk, pv, shared, ck, cv, G, nw in HEAD:
        call = f"attn_layout({pk}, {pv}, {ck}, {cv}, {G}, {str(shared).lower()}, compiled_rw({ck}, {cv}))"
        groups = 1 if G <= 4 else 2
        region = max((ck - 8 + cv - 8) * 128, 64 * ROW + groups * 1024)
        asserts += [f'static_assert({call}.wave_stride == {region}, "{call}: bytes of a wavefront");',
                    f'static_assert({call}.nw == {nw}, "{call}: wavefronts");',
                    f'static_assert({call}.total <= {LDS}, "{call}: LDS");']
    _syntax_check(tmp_path, "dq_decode.hip", asserts)


def test_per_token_wavefronts(tmp_path):
    asserts = []
    for pk, pv, shared, H, G, chunk, nw in TOKEN:
        groups = 1 if G <= 4 else 2
        fit = lambda n: f"tok_layout({pk}, {pv}, {str(shared).lower()}, {H * G}, {H}, {chunk}, {n}, {groups})"
        region = 2 * 9 * 256 + 64 * ROW + groups * 1024
        asserts += [f'static_assert({fit(nw)}.wave_stride == {region}, "{fit(nw)}: bytes of a wavefront");',
                    f'static_assert({fit(nw)}.total <= {LDS}, "{fit(nw)}: LDS");',
                    f'static_assert(tok_waves({groups}) == {nw} || {fit(nw + 1)}.total > {LDS}, "{fit(nw + 1)}");']
    _syntax_check(tmp_path, "dq_token.hip", asserts)
