"""The host rules that choose a kernel, compiled from the library's source: at
the shapes where both choices were timed, the rule takes the faster one."""
import os
import subprocess

import pytest

ROOT = os.path.join(os.path.dirname(__file__), "..")
SRC = os.path.join(ROOT, "paper_2609_09721_amd", "csrc", "efq_attn.hip")
EFQ, EXPQ, LUT, EXPQ6 = 0, 1, 2, 4


def _function(src, head):
    at = src.index(head)
    return src[at: src.index("\n}\n", at) + 3]


@pytest.fixture(scope="module")
def use_half(tmp_path_factory):
    tmp = tmp_path_factory.mktemp("dispatch")
    (tmp / "d.cpp").write_text("""#include <cstdlib>
#include <cstdio>
#include "efq_attn.h"
constexpr int kCUs = 256, kQTile = 256;
""" + _function(open(SRC).read(), "bool use_half(") + """
int main(int, char** v) {
  auto n = [&](int i) { return atoi(v[i]); };
  efq_shape s = {n(1), n(2), n(3), n(4), n(5), n(6)};
  printf("%d", (int)use_half(&s, n(7), n(8), n(9)));
}
""")
    subprocess.run(["g++", "-O1", "-I", os.path.join(ROOT, "include"), "-o", str(tmp / "d"), str(tmp / "d.cpp")],
                   check=True)

    def call(shape, causal, kind, q8=0):
        args = [str(x) for x in (*shape, causal, kind, q8)]
        return subprocess.run([str(tmp / "d"), *args], capture_output=True, text=True, check=True).stdout == "1"
    return call


@pytest.mark.parametrize("shape,causal,kind,q8,half", [
    # few queries: unshared keys streamed from HBM by less than one workgroup a CU
    ((4, 16, 30000, 24, 24, 128), 0, EFQ, 0, False), ((2, 100, 30000, 24, 24, 128), 0, EFQ, 0, False),
    ((4, 16, 30000, 24, 24, 128), 0, LUT, 0, True), ((4, 16, 30000, 24, 24, 128), 0, EFQ, 1, True),
    ((8, 16, 12000, 24, 24, 128), 0, EFQ, 0, True), ((4, 16, 6678, 24, 24, 128), 0, EFQ, 0, True),
    ((4, 16, 30000, 32, 8, 128), 0, EFQ, 0, True), ((4, 16, 30000, 16, 16, 64), 0, EFQ, 0, True),
    # non-causal, one round of eight-wave workgroups that half workgroups share CUs in
    ((2, 1500, 1500, 12, 12, 64), 0, LUT, 0, False), ((2, 1500, 1500, 12, 12, 64), 0, EFQ, 0, True),
    ((2, 1500, 1500, 12, 12, 64), 0, EXPQ, 0, True), ((2, 1500, 1500, 12, 12, 64), 0, LUT, 1, True),
    ((1, 1500, 1500, 24, 24, 128), 0, EXPQ, 0, False), ((1, 1500, 1500, 24, 24, 128), 0, EXPQ6, 0, False),
    ((1, 1500, 1500, 24, 24, 128), 0, EFQ, 0, True), ((1, 1500, 1500, 24, 24, 128), 0, EXPQ, 1, True),
    ((1, 2048, 1100, 32, 8, 128), 0, LUT, 0, True), ((1, 2500, 1500, 24, 24, 128), 0, LUT, 0, False),
    ((1, 1800, 800, 24, 24, 128), 0, LUT, 0, True), ((1, 4000, 1500, 24, 24, 128), 0, EXPQ, 0, True),
    ((1, 1024, 1536, 4, 4, 128), 0, EXPQ, 0, True), ((1, 32760, 2048, 24, 24, 128), 0, EFQ, 0, False),
])
def test_use_half(use_half, shape, causal, kind, q8, half):
    assert use_half(shape, causal, kind, q8) == half
