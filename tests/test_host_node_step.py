"""The trace kernel's node step, compiled for the host: what it takes of a node's four slots."""
import subprocess

import pytest

from paper_2310_03505_amd import build as B

# A chain of nodes, each with one child (the last one a leaf) and three empty
# slots, walked as k_trace walks it: the children of a visited node are those
# that node4_child keeps, all but the nearest go on the stack, leaves into
# the ring.
PROGRAM = r"""
#include <hip/hip_runtime.h>
#include <cstdio>
#include <cstring>
#include <cstdlib>
#include <vector>
#include "rr_internal.h"
using namespace rr;

int main(int argc, char** argv) {
  const int n = atoi(argv[1]);
  const double size = atof(argv[2]), dist = atof(argv[3]);
  const double dir[3] = {atof(argv[4]), atof(argv[5]), atof(argv[6])};
  std::vector<Node4> nodes((size_t)n);
  for (int i = 0; i < n; ++i) {
    // steps as the builders choose them for an extent of `size`
    int e = -126;
    while (size > 255.0 * std::ldexp(1.0, e)) ++e;
    const uint32_t eb[3] = {(uint32_t)(e + 127), (uint32_t)(e + 127), (uint32_t)(e + 127)};
    const float origin[3] = {(float)(-0.5 * size), (float)(-0.5 * size), (float)(-0.5 * size)};
    const uint32_t top = (uint32_t)std::ceil(size / std::ldexp(1.0, e));
    uint32_t qlo[3] = {0, 0, 0}, qhi[3] = {top, top, top};
    const int32_t ref[4] = {i + 1 < n ? i + 1 : leaf_ref_encode(0, 1), kEmpty, kEmpty, kEmpty};
    invert_empty_slots(ref, qlo, qhi);
    pack_node4(nodes[(size_t)i], origin, eb, qlo, qhi, ref);
  }
  float o[3], d[3];
  for (int a = 0; a < 3; ++a) {
    d[a] = (float)dir[a];
    o[a] = (float)(-dist * dir[a]);
  }
  RayBox rb;
  ray_box_setup(o[0], o[1], o[2], d[0], d[1], d[2], rb);
  const RaySigns sg = ray_signs(rb);
  const float tmax = (float)(4.0 * dist), k = ray_scale(tmax), limit = tmax * k * kSlabSlack;
  std::vector<int32_t> stack, ring;
  int32_t cur = 0;
  int visits = 0, empty_met = 0;
  size_t deepest = 0;
  for (;;) {
    if ((uint32_t)cur >= (uint32_t)n) {
      if (stack.empty()) break;
      cur = stack.back();
      stack.pop_back();
    }
    const Node4& nd = nodes[(size_t)std::min((uint32_t)cur, (uint32_t)n - 1u)];
    if (++visits > 4 * n + 100) break;
    float tn[4], tf[4];
    node4_slabs(nd.w0, nd.w1, nd.w2, o[0], o[1], o[2], rb.ix * k, rb.iy * k, rb.iz * k, sg, tn, tf);
    for (int j = 1; j < 4; ++j) empty_met += tn[j] <= tf[j] * kSlabSlack && tn[j] <= limit;
    double key[4];
    uint32_t leaf[4];
    const int32_t ref[4] = {nd.w3.x, nd.w3.y, nd.w3.z, nd.w3.w};
    for (int j = 0; j < 4; ++j) {
      const ChildTest c = node4_child(ref[j], tn[j], tf[j], limit);
      const uint64_t bits = (uint64_t)c.key << 32 | (uint32_t)ref[j];
      std::memcpy(&key[j], &bits, 8);
      leaf[j] = c.leaf;
    }
    cur = kEmpty;
    double best = INFINITY;
    for (int j = 0; j < 4; ++j) {
      if ((int32_t)leaf[j] < 0 && ref[j] != kEmpty) ring.push_back(ref[j]);
      if (std::signbit(key[j])) continue;
      if (cur != kEmpty) {
        stack.push_back(key[j] < best ? cur : ref[j]);
        if (key[j] < best) { best = key[j]; cur = ref[j]; }
      } else {
        best = key[j];
        cur = ref[j];
      }
    }
    deepest = std::max(deepest, stack.size());
  }
  printf("%d %d %zu %zu %d\n", visits, empty_met, deepest, ring.size(), ring.empty() ? 0 : (int)(ring[0] == leaf_ref_encode(0, 1)));
  return 0;
}
"""


@pytest.fixture(scope="module")
def walk(tmp_path_factory):
    d = tmp_path_factory.mktemp("node_step")
    src, exe = d / "walk.cpp", d / "walk"
    src.write_text(PROGRAM)
    flags = [f for f in B.FLAGS if not f.startswith("--offload-arch")]
    r = subprocess.run([B.HIPCC, "--offload-host-only", *flags, "-O1", "-I", B.CSRC, str(src), "-o", str(exe)],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr

    def run(*args):
        out = subprocess.run([str(exe), *map(str, args)], capture_output=True, text=True, check=True, timeout=60)
        return [int(x) for x in out.stdout.split()]
    return run


@pytest.mark.parametrize("n", [1, 2, 7])
@pytest.mark.parametrize("size, dist, far", [(1.0, 3.0, False), (1e-3, 30.0, False), (1e-3, 1e5, True),
                                             (3e-5, 1e3, True), (2.0, 4e7, True)])
def test_empty_slots_are_never_walked(walk, n, size, dist, far):
    """Seen from a million times its size away a node's empty slots pass the
    box test (its slack is relative to the distance); none may be taken for a
    child.  Every node of the chain is visited exactly once, nothing waits on
    the stack, and the one leaf is found."""
    for d in [(0.6, 0.64, 0.48), (-0.8, 0.36, 0.48), (0.36, -0.48, -0.8)]:
        visits, met, deepest, leaves, right = walk(n, size, dist, *d)
        assert (met > 0) == far
        assert (visits, deepest, leaves, right) == (n, 0, 1, 1)
