"""CPU checks of the host rules that choose launch shapes: the rules of the library's headers, compiled here into a
small program, against plain integer arithmetic."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2409_00876_amd", "csrc")


def _compile(tmp_path_factory, name, source):
    d = tmp_path_factory.mktemp(name)
    src, exe = d / f"{name}.cpp", d / name
    src.write_text(source)
    rocm = os.environ.get("ROCM_PATH", "/opt/rocm")
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-D__HIP_PLATFORM_AMD__", "-I", os.path.join(rocm, "include"),
                           "-I", CSRC, str(src), "-o", str(exe)])
    return str(exe)


def _rows(exe, lines):
    out = subprocess.run([exe], input="".join(f"{line}\n" for line in lines), capture_output=True, text=True,
                         check=True).stdout
    return [tuple(int(v) for v in row.split()) for row in out.splitlines()]


@pytest.fixture(scope="module")
def sps_split(tmp_path_factory):
    exe = _compile(tmp_path_factory, "sps_split", r"""
#include <cstdio>
#include "stress.h"
int main() {
  unsigned long long S, m, threads;
  while (scanf("%llu %llu %llu", &S, &m, &threads) == 3) {
    const pgsgd::SpsSplit s = pgsgd::sps_split(S, (uint32_t)m, threads);
    printf("%u %u\n", s.per, s.chunks);
  }
}
""")
    return lambda lines: _rows(exe, lines)


def test_sps_split_covers_every_pair_of_a_step(sps_split):
    # every number of pairs up to the largest 32-bit one, at sizes below and above the grid's 524,288 threads
    threads = 524288
    cases = [(S, m) for S in (1, 2, 3, 100, 14400, 262144, 524287, 524288, 10 ** 9)
             for m in (1, 2, 7, 977, 2 ** 31 - 1, 2 ** 31, 2 ** 31 + 1, 4294200000, 2 ** 32 - 2, 2 ** 32 - 1)]
    got = sps_split([f"{S} {m} {threads}" for S, m in cases])
    assert len(got) == len(cases)
    for (S, m), (per, chunks) in zip(cases, got):
        want = 1 if S >= threads else max(1, min(m, threads // S))
        assert per == -(-m // want), (S, m)
        # chunks * per reaches m, the last chunk is not empty, and chunks of a small graph fit the grid
        assert (chunks - 1) * per < m <= chunks * per, (S, m)
        assert chunks == 1 or S * chunks <= threads, (S, m)
