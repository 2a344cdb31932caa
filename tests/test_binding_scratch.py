"""What the binding asks torch's allocator for (no GPU: the allocation itself is
replaced): nothing that a call cannot use."""
import ctypes

import pytest

BIG = (2, 1, 8192, 32, 8, 128)      # splits


@pytest.fixture
def asked(monkeypatch):
    from paper_2609_09721_amd import binding as B
    sizes = []
    monkeypatch.setattr(B, "_scratch", lambda n, device, stream=None: sizes.append(n))
    return B, sizes


class Q:
    device = "cuda"


def test_split_scratch_only_where_a_call_can_split(asked):
    B, sizes = asked
    sh = B.Shape(*BIG)
    split = [int(B.lib().efq_attn_split_bytes(ctypes.byref(sh), q)) for q in (0, 1)]
    assert min(split) > 0
    for qk8 in (0, 1):
        del sizes[:]
        for causal, kind in ((False, B.PGEN_EFQ), (False, B.PGEN_EXPQ), (True, B.PGEN_EFQ), (False, B.PGEN_NOOP)):
            B._split_scratch(sh, causal, kind, bool(qk8), "cuda", None)
        assert sizes == [split[qk8], split[qk8], 0, 0]
        del sizes[:]
        for causal, kind in ((False, B.PGEN_EFQ), (True, B.PGEN_EFQ), (False, B.PGEN_NOOP)):
            B._workspace(Q, sh, causal, kind, bool(qk8), None, None)
        low = B.vhat_bytes(sh)
        if qk8:
            low += sum(int(f(ctypes.byref(sh))) for f in (B.lib().efq_qhat_bytes, B.lib().efq_khat_bytes))
        assert sizes == [low + split[qk8], low, low]
