"""The host rules that pick a launch's form (ringx_kernels.h), compiled and asked on the CPU: a form is
taken only where it was measured to win."""

import os
import shutil
import subprocess

import pytest

from paper_2507_16697_amd import build as B

ROCM_INCLUDE = "/opt/rocm/include"
pytestmark = pytest.mark.skipif(shutil.which("g++") is None or not os.path.isdir(ROCM_INCLUDE),
                                reason="needs g++ and the HIP headers")

MAIN = r"""
#include <cstdio>
#include "ringx_kernels.h"
int main() {
  using namespace ringx;
  long long kind, d, n, keys;
  while (std::scanf("%lld %lld %lld %lld", &kind, &d, &n, &keys) == 4) {
    const QueryCut c = query_cut(n, keys, kind == 0 ? fwd_cut_rule(d) : dq_cut_rule(d));
    std::printf("%d %d\n", c.ks, c.half ? 1 : 0);
  }
}
"""
PARTIALS_MAIN = r"""
#include <cstdio>
#include "ringx_kernels.h"
int main() {
  using namespace ringx;
  long long n, Nk, R, d;
  while (std::scanf("%lld %lld %lld %lld", &n, &Nk, &R, &d) == 4) {
    const FwdPlan p = fwd_plan(n, Nk, R, d, true);
    std::printf("%d %lld\n", p.cut.ks, (long long)p.rg);
  }
}
"""
DS_MAIN = r"""
#include <cstdio>
#include "ringx_kernels.h"
int main() {
  long long nh, Nq, Nk, R;
  while (std::scanf("%lld %lld %lld %lld", &nh, &Nq, &Nk, &R) == 4)
    std::printf("%d\n", ringx::dq_ds_streams(nh, Nq, Nk, R) ? 1 : 0);
}
"""
TOK_MAIN = r"""
#include <cstdio>
#include "ringx_kernels.h"
int main() {
  long long k, rows, sx, W, x0;
  while (std::scanf("%lld %lld %lld %lld %lld", &k, &rows, &sx, &W, &x0) == 5)
    std::printf("%d\n", ringx::tok_rows_form(k, rows, sx, W, x0).one_row ? 1 : 0);
}
"""
FWD, DQ = 0, 1


def _build(tmp_path, main):
    src, exe = tmp_path / "rules.cpp", tmp_path / "rules"
    src.write_text(main)
    subprocess.run(["g++", "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-I", ROCM_INCLUDE, "-I", B.CSRC,
                    str(src), "-o", str(exe)], check=True, capture_output=True)
    return lambda rows: [tuple(map(int, l.split())) for l in subprocess.run(
        [str(exe)], input="\n".join(" ".join(map(str, r)) for r in rows), text=True, check=True,
        capture_output=True).stdout.splitlines()]


def test_query_cuts(tmp_path):
    ask = _build(tmp_path, MAIN)
    # (kernel, d, workgroups of 256 queries, keys) -> (key streams, half-size workgroups)
    cases = {
        # one round holds the smaller workgroups
        (FWD, 128, 1, 4096): (4, 0), (FWD, 64, 64, 4096): (4, 0), (FWD, 128, 65, 4096): (2, 0),
        (DQ, 128, 128, 4096): (2, 0), (FWD, 128, 129, 4096): (1, 0), (DQ, 128, 256, 4096): (1, 0),
        # a stream owns at least one tile of 64 keys
        (FWD, 128, 1, 255): (2, 0), (FWD, 128, 1, 127): (1, 0), (DQ, 64, 100, 100): (1, 0),
        # ragged rounds at d = 128: only from the key counts on where two streams win
        (FWD, 128, 257, 200): (1, 0), (FWD, 128, 384, 2047): (1, 0), (FWD, 128, 384, 2048): (2, 0),
        (FWD, 128, 385, 8192): (1, 0), (FWD, 128, 576, 4096): (1, 0), (FWD, 128, 640, 16384): (2, 0),
        (FWD, 128, 769, 200): (1, 0), (FWD, 128, 896, 65536): (1, 0),
        (DQ, 128, 257, 200): (2, 0), (DQ, 128, 384, 128): (2, 0), (DQ, 128, 576, 512): (1, 0),
        (DQ, 128, 576, 1024): (2, 0), (DQ, 128, 832, 8192): (1, 0),
        # d = 64: half-size workgroups
        (FWD, 64, 257, 200): (1, 1), (FWD, 64, 385, 200): (1, 0), (FWD, 64, 512, 16384): (1, 1),
        (FWD, 64, 1024, 16385): (1, 0), (DQ, 64, 576, 8192): (1, 1), (DQ, 64, 767, 200): (1, 0),
        (DQ, 64, 768, 4096): (1, 1), (DQ, 64, 768, 4097): (1, 0),
    }
    got = dict(zip(cases, ask(cases)))
    assert got == cases, {k: (got[k], cases[k]) for k in cases if got[k] != cases[k]}


def test_partials_streams_have_tiles(tmp_path):
    """Streams split the chunks of a group one after the other, so what counts is a chunk's length, also
    where a workgroup takes several short chunks."""
    ask = _build(tmp_path, PARTIALS_MAIN)
    rows = [(5, 26416, 208, 128), (14, 9525, 75, 128), (27, 4826, 38, 128), (2, 8000, 4000, 128)]
    rows += [(n, c * R, R, d) for d in (64, 128) for n in (1, 5, 20, 130, 300, 576, 900)
             for R in (1, 2, 3, 8, 100, 700) for c in (1, 40, 64, 127, 128, 5000)]
    for (n, Nk, R, d), (ks, rg) in zip(rows, ask(rows)):
        assert 1 <= rg <= R and ks in (1, 2)
        assert ks == 1 or Nk // R >= 64 * ks, (n, Nk, R, d, ks, rg)


def test_stored_ds_streams(tmp_path):
    ask = _build(tmp_path, DS_MAIN)
    # (query heads, queries, keys, chunks) -> key-stream kernel
    cases = {(1, 100, 32, 1): 1, (2, 4096, 16384, 4): 1, (64, 128, 64, 1): 1, (65, 32, 255, 1): 0,
             (128, 32, 256, 1): 1, (128, 64, 400, 1): 1, (128, 100, 100, 1): 0, (3, 4096, 2000, 2): 0,
             (8, 2048, 512, 1): 0, (1, 16384, 4000, 1): 0, (1, 16384, 16384, 1): 1,
             (4, 4096, 2000, 100): 1, (129, 20, 8000, 1): 0}
    got = dict(zip(cases, (r[0] for r in ask(cases))))
    assert got == cases, {k: got[k] for k in cases if got[k] != cases[k]}


def test_partials_chunk_groups(tmp_path):
    """Chunk groups only where the rounds they save outweigh what every workgroup and chunk costs, and
    counted by the largest group."""
    ask = _build(tmp_path, PARTIALS_MAIN)
    # (workgroups of 256 queries, keys, chunks, d) -> chunk groups
    cases = {(200, 2400, 8, 128): 1, (200, 32000, 8, 128): 8, (640, 12000, 3, 128): 3,
             (1100, 12000, 3, 128): 1, (450, 3600, 8, 128): 1, (640, 16000, 4, 128): 2,
             (900, 3600, 4, 128): 1, (128, 32768, 8, 128): 8, (128, 32768, 8, 64): 8,
             (1100, 12000, 3, 64): 1, (640, 4000, 4, 64): 2, (480, 32768, 8, 128): 1}
    got = dict(zip(cases, (rg for _, rg in ask(cases))))
    assert got == cases, {k: got[k] for k in cases if got[k] != cases[k]}


def test_tokenizer_rows_in_flight(tmp_path):
    ask = _build(tmp_path, TOK_MAIN)

    def rows(C, D, H, k):
        return C * (D // k) * (H // k)

    # (k, filtered rows, cells of a row, field width, first cell) -> one field row in flight
    cases = {(8, rows(2, 64, 64, 8), 640, 640, 0): 0, (4, rows(2, 64, 64, 4), 4096, 4096, 0): 0,
             (8, rows(2, 64, 64, 8), 4096, 4096, 0): 0, (4, rows(4, 512, 512, 4), 512, 512, 0): 0,
             (4, rows(1, 1024, 1024, 4), 1024, 1024, 0): 0,
             (4, rows(4, 1024, 1024, 4), 1024, 1024, 4): 0,
             (4, rows(4, 1024, 1024, 4), 1024, 1024, 0): 1,
             (4, rows(4, 512, 512, 4), 512, 1024, 259): 1,
             (4, rows(4, 512, 512, 4), 768, 1536, 0): 0, (8, rows(4, 512, 512, 8), 512, 1024, 3): 1,
             (8, rows(4, 384, 384, 8), 384, 768, 0): 0, (8, rows(4, 512, 512, 8), 512, 512, 0): 0,
             (8, rows(4, 1024, 1024, 8), 1024, 1024, 3): 0,
             (8, rows(4, 1024, 1024, 8), 1024, 1024, 508): 1,
             (16, rows(4, 512, 512, 16), 512, 1024, 1): 1,
             (16, rows(4, 1024, 1024, 16), 1024, 1024, 0): 0,
             (2, rows(2, 64, 64, 2), 512, 512, 0): 0, (2, rows(4, 512, 512, 2), 512, 512, 0): 1}
    got = dict(zip(cases, (r[0] for r in ask(cases))))
    assert got == cases, {k: got[k] for k in cases if got[k] != cases[k]}
