"""The host rules that choose a launch's shape (launch.hpp), compiled for the
host and called directly: no GPU is needed.  What they must never get wrong
(every row covered once, a workspace that is not overrun), and which side of a
measured line a shape falls on."""

import ctypes
import os
import shutil
import subprocess

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HIPCC = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"

SOURCE = r"""
#include "launch.hpp"
using namespace vidax;
extern "C" void token_rule(int B, int L, int H, int* out) {
  const TokenSplit s = token_split(B, L, H);
  out[0] = s.rows; out[1] = s.nb; out[2] = s.gx; out[3] = s.gy; out[4] = s.gz;
}
extern "C" void bwd_rule(int B, int H, int Lq, int Lk, int cus, size_t max_floats, int lengths, size_t* out) {
  const BwdSplit s = attn_bwd_split(B, H, Lq, Lk, cus, max_floats, lengths != 0);
  out[0] = s.kper; out[1] = s.qsplit; out[2] = s.qper; out[3] = s.part_offset; out[4] = s.floats;
}
"""


@pytest.fixture(scope="module")
def rules(tmp_path_factory):
    if not os.path.exists(HIPCC):
        pytest.skip("hipcc is not available")
    d = tmp_path_factory.mktemp("rules")
    src, lib = d / "rules.cpp", d / "librules.so"
    src.write_text(SOURCE)
    res = subprocess.run([HIPCC, "--offload-arch=gfx950", "--offload-host-only", "-O1", "-std=c++17", "-fPIC", "-shared",
                          "-x", "hip", "-I", os.path.join(ROOT, "paper_2609_18077_amd", "csrc"), str(src), "-o",
                          str(lib)], capture_output=True, text=True, timeout=300)
    assert res.returncode == 0, res.stderr[-4000:]
    return ctypes.CDLL(str(lib))


def _token(rules, B, L, H):
    out = (ctypes.c_int * 5)()
    rules.token_rule(B, L, H, out)
    return list(out)


def _token_shapes():
    rng = np.random.default_rng(61)
    edges = [(1, 1, 1), (1, 16, 40), (1, 40, 5), (2, 40, 5), (5, 40, 3), (1, 901, 11), (2, 901, 13), (64, 520, 1),
             (1, 5120, 24), (1, 5121, 24), (1, 16384, 7), (1, 16385, 7), (33, 8200, 3), (2000, 16, 1), (1, 16, 5000)]
    return edges + [(int(rng.integers(1, 40)), int(np.exp(rng.uniform(0, 11))), int(rng.integers(1, 60)))
                    for _ in range(300)]


def test_token_split_covers_every_row_once(rules):
    """Workgroup (x, y, z): heads x * rows .. of batches z * nb .., every gy-th
    group of 16 tokens.  No share is empty, none is missing."""
    for B, L, H in _token_shapes():
        rows, nb, gx, gy, gz = _token(rules, B, L, H)
        groups = -(-L // 16)
        assert (gx - 1) * rows < H <= gx * rows, (B, L, H)
        assert (gz - 1) * nb < B <= gz * nb, (B, L, H)
        assert 1 <= gy <= min(groups, 1024), (B, L, H)
        assert gy == groups or gx * gz == 1, (B, L, H)  # a strided walk takes all rows
        assert gx == 1 or (rows % 4 == 0 and nb == 1), (B, L, H)
        assert gz <= 65535


def test_token_split_repeats_the_angles_only_where_it_pays(rules):
    """Each share of a token's rows forms the token's angles anew: up to 320
    groups of tokens (a workgroup per compute unit) a share has at most half the
    chain of rows, four at a time; past that it has at least eight rows."""
    for B, L, H in _token_shapes():
        rows, nb, gx, gy, gz = _token(rules, B, L, H)
        if gx * gz == 1:
            continue
        if -(-L // 16) <= 320:
            assert 2 * -(-rows * nb // 4) <= -(-B * H // 4) and gx * gy * gz <= 4096, (B, L, H)
        else:
            assert rows * nb >= 8 and gx * gy * gz <= 2560, (B, L, H)
    assert _token(rules, 1, 15600, 5)[2] == 1     # two shares: 10.1 against 8.2 us
    assert _token(rules, 1, 7800, 12)[2] == 1     # half split, two shares: 13.9 against 11.7 us
    assert _token(rules, 1, 4680, 10)[2] == 1     # eight heads and two: 7.4 against 6.3 us
    assert _token(rules, 1, 8200, 40)[2] == 1     # 12, 12, 12 and 4 heads: 30.1 against 27.9 us
    assert _token(rules, 1, 7800, 40)[2] == 5     # one share: 26.5 against 25.8 us
    assert _token(rules, 1, 7800, 24)[2] == 2     # one share: 18.6 against 18.0 us
    assert _token(rules, 1, 1560, 12)[2] == 3     # one share: 8.2 against 6.4 us


NO_LIMIT = 2 ** 62


def _bwd(rules, B, H, Lq, Lk, max_floats=NO_LIMIT, lengths=False, cus=256):
    out = (ctypes.c_size_t * 5)()
    rules.bwd_rule(B, H, Lq, Lk, cus, ctypes.c_size_t(max_floats), int(lengths), out)
    return list(out)


def _bwd_shapes():
    rng = np.random.default_rng(62)
    return [(int(rng.integers(1, 4)), int(rng.integers(1, 60)), int(np.exp(rng.uniform(0, 11))),
             int(np.exp(rng.uniform(0, 11)))) for _ in range(300)]


def test_bwd_split_fits_its_workspace(rules):
    """Every query tile lies in one run, the partials end within the workspace
    the rule asks for and within 384 MiB, and a call with any smaller workspace
    (down to D alone) takes runs that fit it."""
    for B, H, Lq, Lk in _bwd_shapes():
        tiles, rows, run = -(-Lq // 64), B * H * Lq, 2 * B * H * Lk * 128
        full = _bwd(rules, B, H, Lq, Lk)[4]
        for limit in (NO_LIMIT, full, full - 1, (full + rows) // 2, rows):
            if limit < rows:
                continue
            for lengths in (False, True):
                kper, qsplit, qper, off, floats = _bwd(rules, B, H, Lq, Lk, limit, lengths)
                assert floats <= limit and floats <= full, (B, H, Lq, Lk, limit)
                assert 1 <= qsplit <= 32 and qsplit * qper >= tiles
                assert kper in (128, 256) and (qsplit == 1 or kper == 256)
                if qsplit > 1:
                    assert off % 64 == 0 and off >= rows and floats == off + qsplit * run
                    assert qsplit * run * 4 <= 384 << 20
                else:
                    assert floats == rows


def test_bwd_split_with_a_smaller_workspace_keeps_splitting(rules):
    """A workspace of the size an earlier choice asked for (fewer runs) is used
    as far as it goes, not given up for no split at all."""
    B, H, Lq, Lk = 1, 12, 16384, 77
    run, rows = 2 * B * H * Lk * 128, B * H * Lq
    assert _bwd(rules, B, H, Lq, Lk)[1] == 20
    for s in (2, 8, 16, 19):
        assert s // 2 < _bwd(rules, B, H, Lq, Lk, rows + 64 + s * run)[1] <= s, s


def test_bwd_split_bound_keeps_the_runs_that_pay(rules):
    """Runs on both sides of the bound on the partials."""
    assert _bwd(rules, 1, 3, 23058, 23058)[1] == 5  # 354 MB: 2901 us, two runs 3037
    assert _bwd(rules, 2, 3, 11520, 11520)[1] == 4  # 283 MB: 1527 us, two runs 1557
    assert _bwd(rules, 1, 3, 39167, 39167)[1] == 1  # five runs, 601 MB: 6569 us, unsplit 6508
    assert _bwd(rules, 2, 2, 28000, 28000)[1] == 1  # four runs, 459 MB: 4431 us, unsplit 4381


def test_bwd_key_workgroups(rules):
    """128 or 256 keys a workgroup, on the measured sides of the line."""
    full, half = 256, 128
    assert _bwd(rules, 1, 130, 300, 300)[0] == half   # 2 rounds of either: 61.8 against 53.6 us
    assert _bwd(rules, 1, 100, 300, 600)[0] == half   # 73.2 against 68.9 us
    assert _bwd(rules, 1, 200, 300, 300)[0] == full   # 2 against 3 rounds: 73.0 and 75.8 us
    assert _bwd(rules, 1, 200, 500, 512)[0] == full   # 2 against 4 rounds: 112.6 and 134.3 us
    assert _bwd(rules, 1, 260, 64, 300)[0] == full    # 3 against 4 rounds of one tile: 53.7 and 55.1 us
    assert _bwd(rules, 1, 260, 500, 300)[0] == half   # of eight tiles: 140.6 and 130.9 us
    assert _bwd(rules, 1, 12, 1560, 1560)[:2] == [half, 1]  # runs: 103.8 against 93.9 us
    # lengths of their own: no more rounds than with full workgroups
    assert _bwd(rules, 2, 12, 3000, 3000)[0] == half
    assert _bwd(rules, 2, 12, 3000, 3000, lengths=True)[0] == full
