"""The quantisers of a low-bit call run in one launch where the call is short
and in two where it is long; both must write what the separate entry points
write (the oracle checks those elsewhere), so the outputs are equal bit for bit."""
import pytest
import torch

pytestmark = pytest.mark.gpu


# batch, seq, heads, head_dim: ragged, a single token, the last short call and a long one
@pytest.mark.parametrize("b,s,hq,hkv,D", [(2, 75, 6, 3, 128), (1, 1, 2, 1, 64), (3, 1000, 4, 2, 64),
                                          (1, 6500, 32, 8, 128), (1, 6600, 32, 8, 128)])
def test_one_launch_equals_separate(b, s, hq, hkv, D):
    from paper_2609_09721_amd import binding as B
    print(f"[quant] {(b, s, hq, hkv, D)}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(s)
    q, k, v = (torch.randn((b, s, h, D), generator=g, device="cuda").bfloat16() for h in (hq, hkv, hkv))
    sh = B.shape_of(q, k)
    qh, kh = B.quant_qk(q, k)
    ref = B.attn_fwd_qk8(qh, kh, B.quant_v(v, seq_q=s, heads_q=hq), sh, causal=True)
    n = B.lowbit_workspace_bytes(sh)
    ws = torch.full((n + 256,), 0xA5, dtype=torch.uint8, device="cuda")
    ws = ws[(-ws.data_ptr()) % 256:][:n]
    assert torch.equal(B.attn_fwd_lowbit(q, k, v, causal=True, workspace=ws), ref)
    # Q^ and K^ sit in the workspace in that order, at 256-byte boundaries
    rows = lambda h: b * h * 64 * ((s + 63) // 64)
    at = 0
    for x, h in ((qh, hq), (kh, hkv)):
        codes, scales = rows(h) * D, rows(h) * (D // 32)
        off = (codes + 255) // 256 * 256
        assert torch.equal(ws[at: at + codes], x[:codes])
        assert torch.equal(ws[at + off: at + off + scales], x[off: off + scales])
        at += (x.numel() + 255) // 256 * 256
