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


@pytest.fixture(scope="module")
def local_grids(tmp_path_factory):
    exe = _compile(tmp_path_factory, "local_grids", r"""
#include <cstdio>
#include "local.h"
using namespace pgsgd;
int main() {  // per phase: the cap and the waves that take work on each XCD
  unsigned long long n, paths, S, inflight, resident, scale;
  while (scanf("%llu %llu %llu %llu %llu %llu", &n, &paths, &S, &inflight, &resident, &scale) == 6) {
    const LocalGrids G = local_grids((uint32_t)n, (uint32_t)paths, S, inflight, resident, (uint32_t)scale);
    for (uint32_t ph = 0; ph < kPhases; ++ph) {
      unsigned long long cap = inflight ? inflight : auto_local_waves((uint32_t)n, (uint32_t)paths, S, (LocalPhase)ph,
                                                                     (uint32_t)scale);
      printf("%llu", cap < resident ? cap : resident);
      for (uint32_t x = 0; x < kXcds; ++x) {
        uint32_t blocks = 0;
        for (uint32_t b = x; b < G.blocks[ph]; b += kXcds)
          blocks += b / kXcds < (x < G.hi_xcds[ph] ? G.quota_hi[ph] : G.quota_lo[ph]);
        printf(" %u", blocks * G.threads[ph] / 64);
      }
      printf("\n");
    }
  }
}
""")
    return lambda lines: _rows(exe, lines)


def test_window_grids_stay_within_their_wave_caps(local_grids):
    # few and many paths over the range where the XCDs share unequally and beyond; single layouts, batches, a caller's
    # cap
    cases = []
    for n in (1, 2047, 4096, 20000, 32767, 32768, 33000, 40961, 49000, 50000, 60000, 65000, 65535, 65536, 300000,
              10 ** 7):
        for paths, steps in ((1, n), (1, 3 * n), (4, n), (4, 60 * n), (24, 20 * n), (90, 80 * n)):
            for scale in (0, 1, 2):
                cases.append((n, paths, steps, 0, 6144, scale))
            cases.append((n, paths, steps, 37, 6144, 0))
        cases.append((n, 24, 20 * n, 0, 100, 0))
    got = local_grids([" ".join(map(str, c)) for c in cases])
    assert len(got) == 3 * len(cases)
    for k, row in enumerate(got):
        case, cap, xcds = cases[k // 3], row[0], row[1:]
        assert 1 <= sum(xcds) <= max(1, cap), (case, row)
        if cap >= 32:
            assert min(xcds) >= 1, (case, row)  # every XCD works on its own run
            assert 2 * sum(xcds) > cap, (case, row)  # and the cap is used


def test_few_paths_take_few_waves(local_grids):
    # S / 2048 waves up to seven steps a node, or n / 2048, in every phase, alone and in a batch; with many paths the
    # cap does not bind
    cases = [(n, paths, paths * n // 2, 0, 6144, scale) for n in (36864, 52000, 84000, 340000, 3000000)
             for paths in (1, 2, 3, 6, 10, 14, 24, 40) for scale in (0, 2)]
    got = local_grids([" ".join(map(str, c)) for c in cases])
    for k, row in enumerate(got):
        n, paths, S, _, _, scale = cases[k // 3]
        if paths <= 14:
            assert row[0] <= max(n // 2048, S // 2048), (cases[k // 3], row)
        elif scale == 0 and k % 3 == 1:  # uniform partners, S / n = 12 and more
            assert row[0] >= min(n // 64, 1024), (cases[k // 3], row)
