"""The half-workgroup attention kernel (four waves, two workgroups on a CU):
its LDS ring schedule replayed on the CPU, its work order, and on the GPU its
output against the eight-wave kernel's.  Both run the same tile code in the
same order per query, so the outputs must be equal bit for bit; the entry
point that records the probability stage always runs the eight-wave kernel."""
import os
import subprocess

import pytest
import torch

SRC = os.path.join(os.path.dirname(__file__), "..", "paper_2609_09721_amd", "csrc", "efq_attn.hip")

P, KRING, VRING = 2, 3, 4


def test_ring_schedule():
    src = open(SRC).read()
    for line in ("constexpr int kHP = 2; ", "constexpr int kHK = kHP + 1;", "constexpr int kHV = kHP + 2;",
                 "wait_vmem_le((kHP - 1) * LOADS);"):
        assert line in src
    for ntiles in range(1, 20):
        for T in range(1, ntiles + 1):
            # (ring, tile, iteration of the read, iteration of its consumption)
            reads = [("K", j, j, j) for j in range(T)]
            # V~(j) is consumed by M(j+1), or by F right after iteration T-1's barrier
            reads += [("V", j, j, j + 1) for j in range(T)]
            for ring, x, t, _ in reads:
                landed = -1 if x == 0 else x - 1          # iteration whose wait covers tile x
                assert landed < t
            for x in range(P, ntiles + P):                # streamed in iteration x - P
                for ring, depth in (("K", KRING), ("V", VRING)):
                    last = max((c for r, y, _, c in reads if r == ring and y == x - depth), default=-1)
                    # consumed before the barrier of an earlier iteration; F of
                    # a wave that is done runs before its next barrier
                    assert last < x - P or (ring == "V" and x - depth == T - 1 and last <= x - P), (ring, x)


@pytest.mark.parametrize("B,Hq,Hkv,nqt", [(1, 32, 8, 16), (2, 32, 8, 8), (4, 12, 12, 10), (8, 8, 1, 1),
                                          (1, 8, 2, 3), (1, 16, 16, 32)])
def test_spread_order_visits_every_item_once(B, Hq, Hkv, nqt):
    # map_work with `spread`: a bijection of the grid onto (batch, head, tile)
    src = open(SRC).read()
    assert "if (i >= kXcdCUs) i = kXcdCUs + items - 1 - i;" in src
    total = B * Hq * nqt
    assert total <= 512 and B * Hq % 8 == 0
    items = total // 8
    heads = items // nqt
    seen = set()
    for n in range(total):
        i = n >> 3
        if i >= 32:
            i = 32 + items - 1 - i
        bh = (n & 7) * heads + i % heads
        seen.add((bh // Hq, bh % Hq, nqt - 1 - i // heads))
    assert len(seen) == total
    assert all(0 <= b < B and 0 <= q < nqt for b, _, q in seen)


def _function(src, head):
    at = src.index(head)
    return src[at: src.index("\n}\n", at) + 3]


# batch, heads, key/value heads, query tiles: every order, on both sides of 256
# and 512 workgroups, heads and workgroups that divide by the 8 XCDs and not
GRIDS = [(1, 32, 8, 16), (1, 24, 24, 12), (1, 12, 12, 21), (1, 12, 12, 32), (3, 12, 12, 9), (1, 1, 1, 257),
         (1, 2, 2, 235), (1, 20, 4, 19), (1, 12, 12, 47), (11, 12, 12, 5), (1, 4, 4, 128), (1, 32, 8, 17),
         (1, 9, 3, 1), (7, 1, 1, 3)]


def test_every_work_order_visits_every_item_once(tmp_path):
    """map_work and work_order themselves, compiled for the host: a bijection
    of the grid onto (batch, head, tile); workgroups that are handed out
    together with the longest are the shortest."""
    src = open(SRC).read()
    prog = tmp_path / "order.cpp"
    prog.write_text("""#include <cstdio>
#include <cstdlib>
#define __device__
#define __forceinline__ inline
constexpr int kXcdCUs = 32, kCUs = 8 * kXcdCUs;
struct { int x; } blockIdx, gridDim;
struct AttnArgs { int B, Hq, Hkv, nqt, xcd_remap, spread; };
template <bool SPREAD>
""" + _function(src, "__device__ __forceinline__ void map_work(") + _function(src, "int work_order(") + """
int main(int, char** v) {
  AttnArgs a;
  a.B = atoi(v[1]); a.Hq = atoi(v[2]); a.Hkv = atoi(v[3]); a.nqt = atoi(v[4]);
  gridDim.x = a.B * a.Hq * a.nqt;
  a.xcd_remap = gridDim.x % 8 == 0;
  a.spread = atoi(v[5]) ? work_order(gridDim.x, (long)a.B * a.Hq) : 0;
  for (blockIdx.x = 0; blockIdx.x < gridDim.x; ++blockIdx.x) {
    int b, hq, qt;
    map_work<true>(a, b, hq, qt);
    printf("%d %d %d\\n", b, hq, qt);
  }
}
""")
    exe = tmp_path / "order"
    subprocess.run(["g++", "-O1", "-o", str(exe), str(prog)], check=True)
    for grid in GRIDS:
        b, hq, _, nqt = grid
        total = b * hq * nqt
        for causal in (0, 1):
            out = subprocess.run([str(exe), *map(str, grid), str(causal)], capture_output=True, text=True, check=True)
            items = [tuple(map(int, line.split())) for line in out.stdout.splitlines()]
            assert sorted(items) == [(x, y, z) for x in range(b) for y in range(hq) for z in range(nqt)], grid
            if causal and (total <= 512 and b * hq % 8 or total > 512 and total % 8):
                by_length = sorted((z for _, _, z in items), reverse=True)
                order = [z for _, _, z in items]
                if total <= 512:
                    order[256:] = order[256:][::-1]
                assert order == by_length, grid


@pytest.fixture(scope="module")
def B():
    from paper_2609_09721_amd import binding
    binding.lib()
    assert torch.cuda.is_available(), "no GPU"
    return binding


SHAPES = [  # batch, seq_q, seq_k, heads, head_dim, causal: all inside use_half
    (1, 1, 1, (2, 1), 64, False), (1, 1, 700, (4, 4), 128, False), (2, 127, 65, (8, 2), 128, False),
    (1, 128, 128, (8, 8), 64, True), (1, 129, 129, (8, 2), 128, True), (3, 300, 300, (8, 8), 128, True),
    (1, 600, 449, (3, 1), 64, False), (1, 1037, 1037, (16, 2), 128, True),
    # causal, by length: 257 to 512 workgroups, heads that divide over the XCDs
    # and that do not, and more workgroups than are resident, not a multiple of 8
    (1, 2048, 2048, (32, 8), 128, True), (1, 1500, 1500, (24, 8), 64, True), (3, 1100, 1100, (12, 4), 128, True),
    (1, 2500, 2500, (20, 4), 64, True), (11, 600, 600, (12, 4), 64, True),
    # more workgroups than the chip holds: O leaves as whole rows, through LDS
    (9, 257, 257, (20, 4), 64, True), (9, 130, 100, (32, 8), 128, False),
]


@pytest.mark.gpu
@pytest.mark.parametrize("shape", SHAPES)
@pytest.mark.parametrize("kind", ["efq", "lut", "expq", "expq6"])
def test_equals_eight_wave_kernel(B, shape, kind):
    b, sq, sk, (hq, hkv), D, causal = shape
    print(f"[half] {shape} {kind}", flush=True)
    g = torch.Generator().manual_seed(sq * 7 + sk)
    q, k, v = (torch.randn(s, generator=g).bfloat16().cuda()
               for s in ((b, sq, hq, D), (b, sk, hkv, D), (b, sk, hkv, D)))
    vh = B.quant_v(v, seq_q=sq, heads_q=hq)
    assert torch.equal(B.attn_fwd_vhat(q, k, vh, causal=causal, kind=kind),
                       B.attn_fwd_dump(q, k, vh, causal=causal, kind=kind)[0])
    sh = B.shape_of(q, k)
    qh, kh = B.quant_qk(q, k)
    assert torch.equal(B.attn_fwd_qk8(qh, kh, vh, sh, causal=causal, kind=kind),
                       B.attn_fwd_qk8_dump(qh, kh, vh, sh, causal=causal, kind=kind)[0])
