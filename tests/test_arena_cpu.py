"""The activation arena's planner on the bottleneck ResNets, compiled for the host.

Steps are the models' layers with the fused bottleneck units that the runtime forms (3x3 +
expansion + next reduction).  A unit reads its inputs while it writes all of its outputs, so no
two tensors that a launch touches may overlap, and every tensor that something reads must free
its range: the arena stays within an eighth of the plan without units.
"""
import os
import subprocess

import pytest

from workloads import CONV2D, MAXPOOL2D
from workloads import specs as sp

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_1804_06087_amd", "csrc")

DRIVER = r"""
#include <cstdio>
#include "arena.h"
int main() {
  int n, tensors;
  if (std::scanf("%d %d", &n, &tensors) != 2) return 1;
  std::vector<rafiki::ArenaStep> s(n);
  for (auto& x : s)
    if (std::scanf("%d %d %d %zu %zu %d", &x.in[0], &x.in[1], &x.out, &x.out_bytes, &x.scratch_bytes, &x.last) != 6) return 1;
  const rafiki::ArenaPlan p = rafiki::plan_arena(s, tensors);
  std::printf("%zu", p.bytes);
  for (auto& x : s) std::printf(" %zu", p.off[x.out]);
  for (size_t o : p.scratch) std::printf(" %zu", o);
}
"""


@pytest.fixture(scope="module")
def plan(tmp_path_factory):
    d = tmp_path_factory.mktemp("arena")
    (d / "driver.cpp").write_text(DRIVER)
    exe = str(d / "driver")
    subprocess.run(["g++", "-std=c++17", "-O1", "-I", CSRC, str(d / "driver.cpp"), "-o", exe], check=True)

    def run(steps):
        """steps: (in, in2, out, bytes, scratch, last); (arena bytes, offsets, scratch offsets)."""
        text = f"{len(steps)} {len(steps)}\n" + "\n".join(" ".join(map(str, s)) for s in steps)
        out = [int(v) for v in subprocess.run([exe], input=text, capture_output=True, text=True, check=True).stdout.split()]
        return out[0], out[1:1 + len(steps)], out[1 + len(steps):]
    return run


def steps_of(spec, n, units):
    """One step per layer; units: with the spans of fused bottleneck launches."""
    L = spec.layers
    shapes, steps = {-1: spec.input_shape}, []
    for i, lay in enumerate(L):
        c, h, w = (tuple(shapes[lay.input]) + (1, 1))[:3]
        if lay.op in (CONV2D, MAXPOOL2D):
            shapes[i] = (lay.c_out, (h + 2 * lay.pad - lay.kh) // lay.stride + 1, (w + 2 * lay.pad - lay.kw) // lay.stride + 1)
        else:
            shapes[i] = (lay.c_out, 1, 1)
        c, h, w = shapes[i]
        steps.append([lay.input, lay.input2, i, 0 if i == len(L) - 1 else n * h * w * c * 2, 0, i])
    covered = set()
    for i, lay in enumerate(L):
        if not (units and lay.op == CONV2D and lay.input2 >= 0 and lay.kh == 1 and lay.c_in in (64, 128, 256)):
            continue
        first = i - 1 if i - 1 not in covered and L[i - 1].kh == 3 and L[i - 1].stride == 1 and lay.input == i - 1 else i
        last = i + 1 if L[i + 1].op == CONV2D and L[i + 1].input == i and L[i + 1].kh == 1 and L[i + 1].c_out == lay.c_in else i
        if first < last:
            for k in range(first, last + 1):
                steps[k][5] = last
                covered.add(k)
    return [tuple(s) for s in steps]


def check_disjoint(steps, off):
    """Tensors whose lives meet, from a launch's first step to its last, lie apart."""
    first = {}
    for k, s in enumerate(steps):
        first.setdefault(s[5], k)
    life = {}
    for a, b, o, _, _, last in steps:
        for t in (a, b, o):
            if t >= 0 and steps[t][3]:
                lo, hi = life.get(t, (last, last))
                life[t] = (min(lo, first[last]), max(hi, last))
    for t, (a0, a1) in life.items():
        for u, (b0, b1) in life.items():
            if t < u and a0 <= b1 and b0 <= a1:
                assert off[t] + steps[t][3] <= off[u] or off[u] + steps[u][3] <= off[t], (t, u)


@pytest.mark.parametrize("builder", [sp.resnet50, sp.resnet101])
def test_fused_units_return_their_inputs(plan, builder):
    spec, n = builder(), 256
    apart, _, _ = plan(steps_of(spec, n, False))
    steps = steps_of(spec, n, True)
    spans = {s[5] for i, s in enumerate(steps) if s[5] > i}
    assert len(spans) > 10
    fused, off, _ = plan(steps)
    check_disjoint(steps, off)
    assert fused <= apart * 9 // 8, (fused, apart)


def test_small_plans(plan):
    # a unit (steps 1-3) over x = 0: nothing that it touches overlaps; what follows reuses it all
    unit = [(-1, -1, 0, 1000, 0, 0), (0, -1, 1, 1000, 0, 3), (1, 0, 2, 4000, 0, 3), (2, -1, 3, 1000, 0, 3),
            (3, 2, 4, 2000, 0, 4), (4, -1, 5, 0, 0, 5)]
    total, off, _ = plan(unit)
    check_disjoint(unit, off)
    assert off[4] < 1024 * 2                     # the ranges of 0 and 1, free again
    # scratch lies apart from its own step's output and is free after it
    _, off, scratch = plan([(-1, -1, 0, 512, 4096, 0), (0, -1, 1, 4096, 0, 1)])
    assert scratch[0] == 0 and off[0] == 4096 and off[1] == 0
    # a tensor that nothing reads is free after the step that writes it
    _, off, _ = plan([(-1, -1, 0, 512, 0, 0), (-1, -1, 1, 512, 0, 1)])
    assert off[1] == off[0]
