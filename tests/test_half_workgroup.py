"""The half-workgroup attention kernel (four waves, two workgroups on a CU):
its LDS ring schedule replayed on the CPU, its work order, and on the GPU its
output against the eight-wave kernel's.  Both run the same tile code in the
same order per query, so the outputs must be equal bit for bit; the entry
point that records the probability stage always runs the eight-wave kernel."""
import os

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
