"""The host rules that choose a kernel, compiled from the library's source: at
the shapes where both choices were timed, the rule takes the faster one."""
import os
import re
import subprocess

import pytest

ROOT = os.path.join(os.path.dirname(__file__), "..")
SRC = os.path.join(ROOT, "paper_2609_09721_amd", "csrc", "efq_attn.hip")
EFQ, EXPQ, LUT, EXPQ6 = 0, 1, 2, 4


def _function(src, head):
    at = src.index(head)
    return src[at: src.index("\n}\n", at) + 3]


def _constants(src, *names):
    return "".join(re.search(rf"^constexpr \w+ {n} = .*?;", src, flags=re.M).group(0) + "\n" for n in names)


@pytest.fixture(scope="module")
def rules(tmp_path_factory):
    """rules(shape, causal, kind, q8) -> (use_half, the split's chunks and scratch bytes)."""
    tmp = tmp_path_factory.mktemp("dispatch")
    src = open(SRC).read()
    at = src.index("struct SplitPlan {")
    (tmp / "d.cpp").write_text("""#include <algorithm>
#include <cmath>
#include <cstdlib>
#include <cstdio>
#include <cstring>
#include "efq_attn.h"
constexpr int kQTile = 256;
size_t round256(size_t n) { return (n + 255) & ~(size_t)255; }
""" + _constants(src, "kXcdCUs", "kCUs", "kBc", "kSWaves", "kSRows", "kSItems", "kSplitScores", "kSplitSums")
        + _function(src, "bool use_half(") + src[at: src.index("};", at) + 3] + _function(src, "SplitPlan split_plan(") + """
int main(int, char** v) {
  auto n = [&](int i) { return atoi(v[i]); };
  efq_shape s = {n(1), n(2), n(3), n(4), n(5), n(6)};
  const SplitPlan p = split_plan(&s, n(9), n(8));
  printf("%d %d %zu", (int)use_half(&s, n(7), n(8), n(9)), p.bytes ? p.nch : 0, p.bytes);
}
""")
    subprocess.run(["g++", "-O1", "-I", os.path.join(ROOT, "include"), "-o", str(tmp / "d"), str(tmp / "d.cpp")],
                   check=True)

    def call(shape, causal, kind, q8=0):
        args = [str(x) for x in (*shape, causal, kind, q8)]
        out = subprocess.run([str(tmp / "d"), *args], capture_output=True, text=True, check=True).stdout
        return tuple(map(int, out.split()))
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
def test_use_half(rules, shape, causal, kind, q8, half):
    assert rules(shape, causal, kind, q8)[0] == half


@pytest.mark.parametrize("split,qk8,shapes", [
    # more than 32 rows: every column tile reads K again; timed unsplit / split (us)
    (False, 0, [(8, 24, 8000, 32, 8, 128),      # 111 / 146
                (8, 32, 8000, 32, 8, 128),      # 111 / 132
                (32, 24, 2000, 32, 8, 128),     # 102 / 125
                (64, 32, 4096, 32, 8, 128),     # 381 / 575
                (8, 128, 8000, 12, 12, 64),     # 85 / 142
                (32, 32, 2000, 16, 4, 64)]),    # 28.8 / 38.2
    (False, 1, [(8, 24, 2000, 32, 8, 128),      # 26.5 / 36.1
                (32, 32, 700, 32, 8, 128),      # 30.3 / 54.3
                (16, 24, 8000, 32, 8, 128),     # 125 / 155
                (128, 32, 4096, 32, 8, 128)]),  # 526 / 950
    (True, 0, [(1, 16, 32768, 32, 8, 128),      # 380 / 52
               (4, 32, 8000, 32, 8, 128),       # 102 / 68
               (16, 16, 8000, 32, 8, 128),      # 198 / 166
               (4, 128, 8000, 12, 12, 64),      # 79.4 / 69.3
               (96, 16, 4096, 16, 4, 64)]),     # 169 / 132
    (True, 1, [(8, 32, 8000, 32, 8, 128),       # 87.4 / 74.4
               (16, 16, 2000, 32, 8, 128),      # 33.2 / 32.2
               (16, 32, 8000, 16, 4, 64)]),     # 76.7 / 39.7
    # one column tile, from eight chunks down to one, whose heads share K
    (True, 0, [(64, 1, 4096, 32, 8, 128),       # 379 / 176
               (128, 8, 4096, 32, 8, 128),      # 739 / 547
               (256, 1, 4096, 32, 8, 128),      # 1473 / 818
               (512, 1, 1024, 32, 8, 128),      # 800 / 414
               (512, 1, 4096, 16, 4, 64)]),     # 864 / 510
    # or do not
    (False, 0, [(64, 1, 2048, 64, 64, 128), (16, 1, 8192, 24, 24, 128)]),
    (False, 1, [(237, 1, 740, 12, 12, 64),      # 68.4 / 106
                (188, 3, 4820, 12, 12, 64),     # 291 / 469
                (36, 1, 9502, 12, 12, 64)]),    # five chunks for eight waves: 111 / 150
    (True, 1, [(46, 1, 6450, 12, 12, 64)]),     # four for four: 126 / 115
    # a full chip: column tiles against heads of a group
    (True, 0, [(365, 6, 3535, 32, 4, 128), (100, 12, 2648, 64, 8, 128)]),        # 1708 / 871, 736 / 522
    (False, 0, [(65, 18, 7499, 32, 8, 128), (110, 31, 1741, 32, 8, 128)]),       # 726 / 891, 298 / 488
])
def test_split_only_where_it_is_faster(rules, split, qk8, shapes):
    for shape in shapes:
        assert (rules(shape, 0, EFQ, qk8)[1] > 0) == split, shape


SHAPES_OF_STAGES = [(b, sq, sk, *h) for b in (1, 8, 40) for sq in (1, 9, 30, 64) for sk in (900, 5000)
                    for h in ((32, 8, 128), (16, 4, 64), (24, 24, 128))]


def test_split_by_stage(rules):
    # timed unsplit / split (us)
    for shape, q8 in (((1, 10, 1259, 32, 8, 128), 0), ((1, 56, 1056, 16, 8, 64), 1), ((17, 6, 669, 32, 4, 128), 1)):
        assert rules(shape, 0, EXPQ6, q8)[1] > 0, shape          # 23.1 / 17.0, 16.7 / 12.0, 28.1 / 19.1
    # three chunks for four waves: EFQ 46.1 / 49.4, exp-then-quantize 58.1 / 51.0
    assert rules((85, 1, 2000, 8, 8, 64), 0, EFQ, 1)[1] == 0 and rules((85, 1, 2000, 8, 8, 64), 0, EXPQ, 1)[1] == 3
    # the scratch query is the plan of the stage that splits wherever another does
    for shape in SHAPES_OF_STAGES:
        for q8 in (0, 1):
            e, l, x, x6 = (rules(shape, 0, k, q8)[2] for k in (EFQ, LUT, EXPQ, EXPQ6))
            assert e in (0, l) and l in (0, x) and x == x6, shape


def test_shapes_of_the_split_tests_split(rules):
    from test_split_keys import SHAPES
    chunks = set()
    for b, sq, sk, (hq, hkv), D in SHAPES:
        for kind in (EFQ, LUT, EXPQ, EXPQ6):
            for q8 in (0, 1):
                n = rules((b, sq, sk, hq, hkv, D), 0, kind, q8)[1]
                assert n > 0, (b, sq, sk, hq, hkv, D, kind, q8)
                chunks.add(min(n, 4))
    assert chunks == {1, 2, 3, 4}


def test_split_scratch_is_bounded(rules):
    """256 MiB of scores and 256 MiB of maxima and partial sums; and every launch
    of the split below 2^32 threads, whatever the batch."""
    most = 0
    for batch in (1, 64, 256, 1024, 4096, 16384, 1 << 17, 1 << 20, 1 << 23):
        for sq, sk, hq, hkv, D in ((1, 4096, 32, 8, 128), (8, 1024, 32, 8, 128), (5, 100, 64, 8, 128),
                                   (32, 4096, 32, 8, 128), (1, 120000, 64, 8, 128), (16, 700, 32, 4, 64)):
            for q8 in (0, 1):
                nch, n = rules((batch, sq, sk, hq, hkv, D), 0, EXPQ, q8)[1:]
                if n:
                    R = sq * hq // hkv
                    wgs = batch * hkv * -(-nch // 4) * -(-R // 32)
                    assert wgs * 256 < 1 << 32 and batch * hkv * R * D < 1 << 32
                most = max(most, n)
    assert 0 < most <= 512 << 20
