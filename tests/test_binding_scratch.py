"""What the binding asks torch's allocator for (no GPU: the allocation itself is
replaced): nothing that a call cannot use, and nothing in the pool of another
stream than the one the call runs on."""
import contextlib
import ctypes

import pytest
import torch

BIG = (2, 1, 8192, 32, 8, 128)      # splits


@pytest.fixture
def asked(monkeypatch):
    from paper_2609_09721_amd import binding as B
    sizes = []
    monkeypatch.setattr(B, "_scratch", lambda n, stream=None: sizes.append(n))
    return B, sizes


def test_split_scratch_only_where_a_call_can_split(asked):
    B, sizes = asked
    sh = B.Shape(*BIG)
    split = [int(B.lib().efq_attn_split_bytes(ctypes.byref(sh), q)) for q in (0, 1)]
    assert min(split) > 0
    for qk8 in (0, 1):
        del sizes[:]
        for causal, kind in ((False, B.PGEN_EFQ), (False, B.PGEN_EXPQ), (True, B.PGEN_EFQ), (False, B.PGEN_NOOP)):
            B._split_scratch(sh, causal, kind, bool(qk8), None)
        assert sizes == [split[qk8], split[qk8], 0, 0]
        del sizes[:]
        for causal, kind in ((False, B.PGEN_EFQ), (True, B.PGEN_EFQ), (False, B.PGEN_NOOP)):
            B._workspace(sh, causal, kind, bool(qk8), None, None)
        low = B.vhat_bytes(sh)
        if qk8:
            low += sum(int(f(ctypes.byref(sh))) for f in (B.lib().efq_qhat_bytes, B.lib().efq_khat_bytes))
        assert sizes == [low + split[qk8], low, low]


def test_scratch_is_in_the_pool_of_the_calls_stream(monkeypatch):
    """Without a stream the call runs on the current device's current stream,
    so the scratch must not follow the tensors' device; a bare handle has no
    pool, and its call goes on without torch's memory."""
    from paper_2609_09721_amd import binding as B
    made, entered = [], []
    monkeypatch.setattr(torch, "empty", lambda n, dtype=None, device=None: made.append((n, device)) or "t")

    @contextlib.contextmanager
    def on(stream):
        entered.append(stream)
        yield

    monkeypatch.setattr(torch.cuda, "stream", on)
    assert B._scratch(256) == "t" and made == [(256, "cuda")] and not entered

    class Handle:
        cuda_stream = 7

    sh = B.Shape(*BIG)
    assert B._scratch(256, Handle()) is None
    assert B._split_scratch(sh, False, B.PGEN_EFQ, False, Handle()) == (None, 0)
    assert B._workspace(sh, False, B.PGEN_EFQ, False, None, Handle()) == (None, 0)
    assert made == [(256, "cuda")]
