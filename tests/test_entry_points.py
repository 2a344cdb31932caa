"""The C entry points that the binding no longer goes through: efq_attn_fwd and
efq_attn_fwd_expq, and the _ex and lowbit _ex entry points without a workspace,
which take one stream-ordered allocation (with the key split's scratch where few
queries split).  Same kernels as with a workspace, so the outputs are equal."""
import ctypes

import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def B():
    from paper_2609_09721_amd import binding
    binding.lib()
    assert torch.cuda.is_available(), "no GPU"
    return binding


# batch, seq_q, seq_k, heads, head_dim, causal: the smallest workload, a causal
# prompt, cross attention, and few queries that run split (one column tile: V is
# quantised in the attention pass; two column tiles)
@pytest.mark.parametrize("b,sq,sk,heads,D,causal", [
    (1, 256, 256, (1, 1), 64, 0), (2, 300, 300, (8, 2), 128, 1), (1, 200, 77, (4, 4), 128, 0),
    (2, 1, 4200, (8, 2), 128, 0), (1, 16, 9000, (32, 8), 128, 0), (3, 8, 1601, (8, 1), 64, 0)])
def test_without_a_workspace(B, b, sq, sk, heads, D, causal):
    hq, hkv = heads
    print(f"[entry] {(b, sq, sk, heads, D, causal)}", flush=True)
    lib = B.lib()
    g = torch.Generator().manual_seed(sq + sk)
    q, k, v = (torch.randn(s, generator=g).bfloat16().cuda()
               for s in ((b, sq, hq, D), (b, sk, hkv, D), (b, sk, hkv, D)))
    sh = B.shape_of(q, k)
    s, scale, n = ctypes.byref(sh), D ** -0.5, ctypes.c_size_t(0)
    splits = not causal and lib.efq_attn_split_bytes(s, 0) > 0
    assert splits == (sk > 1600)
    ptrs = [B._ptr(t) for t in (q, k, v)]
    ws = torch.empty(int(lib.efq_attn_workspace_bytes(s)), dtype=torch.uint8, device="cuda")
    wl = torch.empty(int(lib.efq_attn_lowbit_workspace_bytes(s)) + 256, dtype=torch.uint8, device="cuda")
    wl = wl[(-wl.data_ptr()) % 256:][: int(lib.efq_attn_lowbit_workspace_bytes(s))]

    def run(f, *args):
        out = torch.full(q.shape, float("nan"), dtype=torch.float32, device="cuda")
        rc = f(*ptrs, scale, causal, *[B._ptr(out) if a is out_slot else a for a in args], B._stream())
        assert rc == B.EFQ_OK, lib.efq_strerror(rc)
        return out

    out_slot = object()
    default = {B.PGEN_EFQ: lib.efq_attn_fwd, B.PGEN_EXPQ: lib.efq_attn_fwd_expq}
    for kind in (B.PGEN_EFQ, B.PGEN_EXPQ, B.PGEN_LUT, B.PGEN_EXPQ6):
        p = B._params(kind, None)
        ref = run(lib.efq_attn_fwd_ex, kind, p, out_slot, s, B._ptr(ws), ws.numel())
        assert torch.equal(run(lib.efq_attn_fwd_ex, kind, p, out_slot, s, None, n), ref)
        if kind in default:      # Mean operating point
            assert torch.equal(run(default[kind], out_slot, s), ref)
        low = run(lib.efq_attn_fwd_lowbit_ex, kind, p, out_slot, s, B._ptr(wl), wl.numel())
        assert torch.equal(run(lib.efq_attn_fwd_lowbit_ex, kind, p, out_slot, s, None, n), low)
        assert torch.isfinite(ref).all() and torch.isfinite(low).all()
        assert float((ref - low).abs().max()) > 0
