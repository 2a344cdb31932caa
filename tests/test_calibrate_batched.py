"""The calibration runs many (tau, h) candidates in one launch and keeps only
sums of squares.  Each objective value must be the relative error of that
candidate's own attention output; both sum fp64 squares of the same fp32
values, so they differ by fp64 rounding of at most n terms (n 2^-53 < 1e-9)."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def B():
    from paper_2609_09721_amd import binding
    binding.lib()
    assert torch.cuda.is_available(), "no GPU"
    return binding


# batch, seq, heads, head_dim, causal, candidates: one query and few rows (the
# smallest workspace), half and eight-wave workgroups, more than one launch
@pytest.mark.parametrize("b,sq,sk,heads,D,causal,nt,nh", [
    (1, 1, 70, (2, 1), 64, False, 9, 8), (1, 130, 130, (8, 2), 128, True, 1, 65),
    (2, 300, 300, (4, 4), 64, True, 3, 3), (1, 1100, 1100, (4, 1), 128, True, 2, 2),
    (1, 257, 900, (2, 2), 64, False, 2, 3),
])
def test_objective_of_each_candidate(B, b, sq, sk, heads, D, causal, nt, nh):
    hq, hkv = heads
    print(f"[rho] {(b, sq, sk, heads, D, causal, nt, nh)}", flush=True)
    g = torch.Generator().manual_seed(sq + sk)
    q, k, v = (torch.randn(s, generator=g).bfloat16().cuda()
               for s in ((b, sq, hq, D), (b, sk, hkv, D), (b, sk, hkv, D)))
    ref = B.attn_fwd(q, k, v, causal=causal, params=(-2.7, 2.1)) + 0.01
    taus = np.linspace(-3.4, -2.2, nt).astype(np.float32)
    hs = np.linspace(1.9, 2.8, nh).astype(np.float32)
    best, rho = B.calibrate(q, k, v, ref, taus, hs, causal=causal)
    want = np.zeros_like(rho)
    r = ref.double()
    for i, tau in enumerate(taus):
        for j, h in enumerate(hs):
            o = B.attn_fwd(q, k, v, causal=causal, params=(tau, h)).double()
            want[i, j] = float((o - r).norm() / r.norm())
    assert np.allclose(rho, want, rtol=1e-9, atol=0)
    i, j = np.unravel_index(int(rho.argmin()), rho.shape)
    assert best == (float(taus[i]), float(hs[j]))
    assert np.array_equal(rho, B.calibrate(q, k, v, ref, taus, hs, causal=causal)[1])
