"""Few queries against many keys, split over the keys: when the split is taken
(host rule and scratch sizes, no GPU), and its output against the unsplit
kernels' on the same inputs.  Codes, scales and maxima are the same, so the two
outputs are the same sums in another order: every partial sum is rounded at
most once per tile, per moved maximum and per merged chunk, which bounds the
difference by (3 tiles + chunks) 2^-24 of the largest value in V~."""
import ctypes

import pytest
import torch

FAKE = ctypes.c_void_p(4096)   # aligned, never dereferenced: validation fails first


@pytest.fixture(scope="module")
def B():
    from paper_2609_09721_amd import binding
    binding.lib()
    return binding


def split_bytes(B, shape, qk8=0):
    return B.lib().efq_attn_split_bytes(ctypes.byref(B.Shape(*shape)), qk8)


def test_scratch_sizes(B):
    lib = B.lib()
    # many rows, few keys, or no head sharing and enough sequences: unsplit
    for shape in ((1, 33, 8192, 32, 8, 128), (1, 1, 256, 32, 8, 128), (16, 1, 8192, 24, 24, 128),
                  (1, 4096, 4096, 32, 8, 128), (1, 129, 32768, 4, 4, 64)):
        assert split_bytes(B, shape) == 0 and split_bytes(B, shape, 1) == 0
        sh = B.Shape(*shape)
        assert lib.efq_attn_workspace_bytes(ctypes.byref(sh)) == B.vhat_bytes(sh)
    for shape in ((1, 1, 4096, 32, 8, 128), (8, 1, 6001, 32, 8, 128), (1, 32, 32768, 32, 8, 128),
                  (1, 128, 4096, 2, 2, 64)):
        sh = B.Shape(*shape)
        n = split_bytes(B, shape)
        assert n > 0 and n % 256 == 0
        assert lib.efq_attn_workspace_bytes(ctypes.byref(sh)) == B.vhat_bytes(sh) + n
        q8 = split_bytes(B, shape, 1)
        assert lib.efq_attn_lowbit_workspace_bytes(ctypes.byref(sh)) == (
            lib.efq_qhat_bytes(ctypes.byref(sh)) + lib.efq_khat_bytes(ctypes.byref(sh)) + B.vhat_bytes(sh) + q8)
    assert split_bytes(B, (1, 1, 4096, 32, 8, 96)) == 0
    # the scratch stays bounded: no scores beyond 256 MiB
    assert max(split_bytes(B, (64, sq, 120000, 64, 8, 128), q) for sq in (1, 2, 4, 16) for q in (0, 1)) < 300 << 20


def test_scratch_arguments(B):
    lib, P = B.lib(), B.Params(-3.06, 2.3)
    sh = B.Shape(1, 1, 4096, 32, 8, 128)
    n = B.vhat_bytes(sh)
    f = lambda ws, b, causal=0: lib.efq_attn_fwd_vhat_ws(FAKE, FAKE, FAKE, n, 0.1, causal, 0, P, FAKE,
                                                         ctypes.byref(sh), ws, b, None)
    assert f(None, 64) == B.EFQ_EWORKSPACE
    assert f(ctypes.c_void_p(4100), 64) == B.EFQ_EINVAL
    assert f(None, 0, causal=1) == B.EFQ_EUNSUPPORTED
    nq, nk = (g(ctypes.byref(sh)) for g in (lib.efq_qhat_bytes, lib.efq_khat_bytes))
    g = lambda ws, b: lib.efq_attn_fwd_qk8_ws(FAKE, nq, FAKE, nk, FAKE, n, 0.1, 0, 0, P, FAKE,
                                              ctypes.byref(sh), ws, b, None)
    assert g(None, 64) == B.EFQ_EWORKSPACE
    assert g(ctypes.c_void_p(4100), 64) == B.EFQ_EINVAL


def _inputs(b, sq, sk, hq, hkv, D, dev="cuda"):
    g = torch.Generator().manual_seed(sq * 31 + sk)
    q, k, v = (torch.randn(s, generator=g) for s in ((b, sq, hq, D), (b, sk, hkv, D), (b, sk, hkv, D)))
    return (q * 1.5).bfloat16().to(dev), k.bfloat16().to(dev), v.bfloat16().to(dev)


def _bound(sk, v):
    tiles = (sk + 63) // 64
    return 4 * tiles * 2.0 ** -24 * 1.5 * float(v.abs().max())


SHAPES = [  # batch, seq_q, seq_k, heads, head_dim: rows 1 .. 128, one key past a tile, chunks of one tile
    (1, 1, 1025, (1, 1), 64), (1, 1, 4096, (32, 8), 128), (2, 1, 3001, (16, 1), 128), (1, 31, 2000, (4, 4), 128),
    (1, 33, 1984, (3, 3), 64), (1, 128, 2111, (2, 2), 128), (3, 8, 1601, (8, 1), 64), (1, 16, 9000, (32, 8), 128),
    # fewer chunks than a workgroup has waves: one, two and three, with stored scores and without
    (256, 1, 129, (32, 8), 128), (256, 1, 129, (64, 8), 64), (130, 4, 200, (64, 8), 128), (90, 2, 257, (32, 8), 64),
    (146, 5, 94, (64, 8), 128),
]


@pytest.mark.gpu
@pytest.mark.parametrize("shape", SHAPES)
@pytest.mark.parametrize("kind", ["efq", "lut", "expq", "expq6"])
def test_equals_unsplit(B, shape, kind):
    b, sq, sk, (hq, hkv), D = shape
    print(f"[split] {shape} {kind}", flush=True)
    lib = B.lib()
    q, k, v = _inputs(b, sq, sk, hq, hkv, D)
    sh = B.shape_of(q, k)
    vh = B.quant_v(v, seq_q=sq, heads_q=hq)
    qh, kh = B.quant_qk(q, k)
    p = B._params(B._kind(kind), None)
    for qk8 in (0, 1):
        assert split_bytes(B, (b, sq, sk, hq, hkv, D), qk8) > 0
        ref = torch.empty(q.shape, dtype=torch.float32, device="cuda")
        if qk8:
            out = B.attn_fwd_qk8(qh, kh, vh, sh, kind=kind)
            rc = lib.efq_attn_fwd_qk8(B._ptr(qh), qh.numel(), B._ptr(kh), kh.numel(), B._ptr(vh), vh.numel(),
                                      D ** -0.5, 0, B._kind(kind), p, B._ptr(ref), ctypes.byref(sh), B._stream())
        else:
            out = B.attn_fwd_vhat(q, k, vh, kind=kind)
            rc = lib.efq_attn_fwd_vhat(B._ptr(q), B._ptr(k), B._ptr(vh), vh.numel(), D ** -0.5, 0, B._kind(kind),
                                       p, B._ptr(ref), ctypes.byref(sh), B._stream())
        assert rc == 0
        assert float((out - ref).abs().max()) <= _bound(sk, v), (qk8, float((out - ref).abs().max()))


@pytest.mark.gpu
def test_entry_points_streams_and_capture(B):
    """The whole-call entry points take the split, with and without a workspace
    and on another stream; a captured call replays to the same output."""
    b, sq, sk, hq, hkv, D = 2, 3, 4200, 8, 2, 128
    q, k, v = _inputs(b, sq, sk, hq, hkv, D)
    sh = B.shape_of(q, k)
    vh = B.quant_v(v, seq_q=sq, heads_q=hq)
    ref = B.attn_fwd_vhat(q, k, vh)
    n = B.lib().efq_attn_workspace_bytes(ctypes.byref(sh))
    ws = torch.empty(n, dtype=torch.uint8, device="cuda")
    assert torch.equal(B.attn_fwd(q, k, v), ref)
    assert torch.equal(B.attn_fwd(q, k, v, workspace=ws), ref)
    small = B.attn_fwd(q, k, v, workspace=ws[: B.vhat_bytes(sh)])      # no room for the scratch: unsplit
    assert float((small - ref).abs().max()) <= _bound(sk, v)
    out = torch.empty_like(ref)
    assert torch.equal(B.attn_fwd_noalloc(q, k, v, out), ref)
    low = B.attn_fwd_lowbit(q, k, v)
    wl = torch.empty(B.lowbit_workspace_bytes(sh) + 256, dtype=torch.uint8, device="cuda")
    off = (-wl.data_ptr()) % 256
    assert torch.equal(B.attn_fwd_lowbit(q, k, v, workspace=wl[off: off + B.lowbit_workspace_bytes(sh)]), low)
    side = torch.cuda.Stream()
    torch.cuda.synchronize()
    outs = [torch.empty_like(ref) for _ in range(8)]
    for o in outs:                                     # calls in flight on two streams at once
        B.attn_fwd_vhat(q, k, vh, out=o, stream=side)
        assert torch.equal(B.attn_fwd_vhat(q, k, vh), ref)
    torch.cuda.synchronize()
    assert all(torch.equal(o, ref) for o in outs)
    graph = torch.cuda.CUDAGraph()
    got = torch.empty_like(ref)
    with torch.cuda.graph(graph):
        B.attn_fwd_vhat(q, k, vh, out=got)
        B.attn_fwd(q, k, v, out=out, workspace=ws)
    for i in range(3):
        got.zero_()
        out.zero_()
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(got, ref) and torch.equal(out, ref), i


@pytest.mark.gpu
def test_stream_given_as_a_bare_handle(B):
    """An object with only a cuda_stream is taken as a stream: calls on it go
    on without torch's memory, unsplit or with the library's own allocation."""
    q, k, v = _inputs(2, 3, 4200, 8, 2, 128)
    sh = B.shape_of(q, k)
    vh = B.quant_v(v, seq_q=3, heads_q=8)
    ref, low = B.attn_fwd_vhat(q, k, vh), B.attn_fwd_lowbit(q, k, v)
    side = torch.cuda.Stream()

    class Handle:
        cuda_stream = side.cuda_stream

    torch.cuda.synchronize()
    out = B.attn_fwd_vhat(q, k, vh, stream=Handle())
    whole = B.attn_fwd(q, k, v, stream=Handle())
    lowbit = B.attn_fwd_lowbit(q, k, v, stream=Handle())
    torch.cuda.synchronize()
    assert float((out - ref).abs().max()) <= _bound(4200, v)
    assert torch.equal(whole, ref) and torch.equal(lowbit, low)


@pytest.mark.gpu
def test_default_workspace(B):
    """Without a workspace the binding takes one from torch's allocator: calls
    in flight on two streams, and the size following the shape."""
    side = torch.cuda.Stream()
    for b, s, hq, hkv, D, causal in ((1, 256, 1, 1, 64, False), (2, 700, 8, 2, 128, True), (1, 65, 4, 4, 64, True)):
        q, k, v = _inputs(b, s, s, hq, hkv, D)
        sh = B.shape_of(q, k)
        ws = torch.empty(B.vhat_bytes(sh), dtype=torch.uint8, device="cuda")
        wl = torch.empty(B.lowbit_workspace_bytes(sh), dtype=torch.uint8, device="cuda")
        for kind, call in (("efq", B.efq_attn_fwd), ("expq", B.efq_attn_fwd_expq)):
            ref = B.attn_fwd(q, k, v, causal=causal, kind=kind, workspace=ws)
            low = B.attn_fwd_lowbit(q, k, v, causal=causal, kind=kind, workspace=wl)
            torch.cuda.synchronize()
            for _ in range(4):
                on_side = call(q, k, v, causal=causal, stream=side, out=torch.empty_like(ref))
                assert torch.equal(call(q, k, v, causal=causal), ref)
                assert torch.equal(B.attn_fwd(q, k, v, causal=causal, kind=kind), ref)
                assert torch.equal(B.attn_fwd_lowbit(q, k, v, causal=causal, kind=kind), low)
                side.synchronize()
                assert torch.equal(on_side, ref)


@pytest.mark.gpu
@pytest.mark.parametrize("shape", [(1, 1, 1025, 32, 8, 128), (2, 5, 2111, 6, 3, 128), (1, 16, 3000, 4, 4, 128)])
@pytest.mark.parametrize("kind", ["efq", "lut", "expq", "expq6"])
def test_whole_call_quantises_v_in_place(B, shape, kind):
    """The whole call's split reads V itself; the values are those of V~."""
    b, sq, sk, hq, hkv, D = shape
    print(f"[split v] {shape} {kind}", flush=True)
    assert split_bytes(B, shape) > 0
    q, k, v = _inputs(b, sq, sk, hq, hkv, D)
    v[:, : sk // 2] *= 2.0 ** -9
    v[:, -33:] = 0                       # blocks without a value, and the ragged end
    assert torch.equal(B.attn_fwd(q, k, v, kind=kind),
                       B.attn_fwd_vhat(q, k, B.quant_v(v, seq_q=sq, heads_q=hq), kind=kind))
