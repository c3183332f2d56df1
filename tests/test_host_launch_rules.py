"""Launch sizes, compiled for the host: how a level's rays are spread over waves."""
import subprocess

import pytest

from paper_2310_03505_amd import build as B

PROGRAM = r"""
#include <cstdio>
#include <cstdlib>
#include "kernels.h"
int main(int argc, char** argv) {
  for (int i = 1; i + 3 < argc; i += 4)
    printf("%u\n", rr::trace_blocks(strtoull(argv[i], nullptr, 10), (uint32_t)atoi(argv[i + 1]),
                                    (uint32_t)atoi(argv[i + 2]),
                                    atoi(argv[i + 3]) ? rr::kSpreadRays : rr::kPackedRays));
  return 0;
}
"""
WAVES = 2  # of a trace block


@pytest.fixture(scope="module")
def blocks(tmp_path_factory):
    d = tmp_path_factory.mktemp("rules")
    src, exe = d / "rules.cpp", d / "rules"
    src.write_text(PROGRAM)
    flags = [f for f in B.FLAGS if not f.startswith("--offload-arch")]
    r = subprocess.run([B.HIPCC, "--offload-host-only", *flags, "-O1", "-I", B.CSRC, str(src), "-o", str(exe)],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr

    def run(calls):
        args = [str(x) for c in calls for x in c]
        out = subprocess.run([str(exe), *args], capture_output=True, text=True, check=True, timeout=60)
        return [int(x) for x in out.stdout.split()]
    return run


@pytest.mark.parametrize("spread", [1, 0])
@pytest.mark.parametrize("n_cu", [1, 32, 64, 128, 256, 304])
def test_trace_blocks_scale_with_the_compute_units(blocks, n_cu, spread):
    """A level is spread over at most one wave per SIMD, four of them a
    compute unit, unless it has more than 32 rays for each, or 64 where idle
    lanes cannot help; every ray has a lane until the grid is full; the grid
    is never exceeded."""
    rays = 32 if spread else 64
    grid = 24 * n_cu // WAVES
    bounds = [0, 1, 7, 8, 9, 31 * n_cu, 32 * n_cu, 32 * n_cu + 1, 128 * n_cu - 1, 128 * n_cu, 128 * n_cu + 1,
              256 * n_cu, 256 * n_cu + 1, 1000 * n_cu, 64 * 24 * n_cu, 10**9, 2**31]
    for bound, got in zip(bounds, blocks([(b, grid, n_cu, spread) for b in bounds])):
        assert 1 <= got <= max(grid, 1)
        waves = max(min(-(-bound // 8), 4 * n_cu), -(-bound // rays))
        assert got == min(max(-(-waves // WAVES), 1), grid)
        assert got == grid or got * WAVES * 64 >= bound
        if bound <= 4 * rays * n_cu:
            assert got * WAVES <= 4 * n_cu
