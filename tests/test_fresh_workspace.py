"""GMLP_FRESH_WORKSPACE: a call on memory nobody has prepared (here filled with
ones) gives the bits of a call on a prepared workspace, on every kernel that
counts arrivals; the calls without a workspace, which run this way on memory
of torch's allocator, can be captured; the fused paths refuse the flag."""
import numpy as np
import pytest
import torch

from paper_2606_26344_amd import gmlp
from paper_2606_26344_amd import inputs as I
from paper_2606_26344_amd import softmax_matmul as smm

A, MB = 0x10000000, 1 << 20
FRESH = gmlp.FRESH_WORKSPACE


def test_flag_matches_the_header():
    assert "#define GMLP_FRESH_WORKSPACE %d" % FRESH in open(gmlp.HEADER).read()


def test_fused_paths_refuse_the_flag():
    lib = gmlp.library()
    args = (A, A + 64 * MB, A + 128 * MB, A + 192 * MB, A + 256 * MB, 4, 256, 512)
    n = gmlp.workspace_size(4, 256, 512)
    for path in (gmlp.PATH_FUSED, gmlp.PATH_FUSED_MFMA, 5):
        assert lib.gmlp_forward_ex(*args, path | FRESH, A + 300 * MB, n, None) == 1
    # Checked as without the flag.
    assert lib.gmlp_forward_ex(*args, FRESH, None, n, None) == 1
    assert lib.gmlp_forward_ex(*args, FRESH, A + 300 * MB, n - 1, None) == 4
    assert lib.gmlp_forward_ex(*args[:5], 9, 256, 512, gmlp.PATH_GEMV | FRESH, A + 300 * MB, n, None) == 2
    buf = __import__("ctypes").create_string_buffer(64)
    assert lib.gmlp_describe(4, 256, 512, FRESH, buf, 64) == 1


def _dirty(n):
    t = torch.full((n + 256,), 0xFF, dtype=torch.uint8, device="cuda")
    return t, (t.data_ptr() + 255) & ~255


# GEMV; streaming tiles with and without splits; ring tiles; pairs; a token
# split with a GEMV rest; large tiles with a tail; split down tiles.
CALLS = [(3, 1032, 2056, "auto"), (8, 264, 520, "gemv"), (16, 264, 520, "auto"), (100, 2056, 1544, "auto"),
         (40, 264, 1032, "mfma"), (100, 264, 16384, "auto"), (515, 1032, 14344, "auto"), (704, 264, 14336, "auto"),
         (300, 1032, 2056, "auto")]


@pytest.mark.gpu
@pytest.mark.parametrize("T,D,F,path", CALLS, ids=["T%dD%dF%d-%s" % c for c in CALLS])
def test_fresh_workspace_gives_the_same_bits(T, D, F, path):
    lib = gmlp.library()
    x, wg, wu, wd = (gmlp.from_bf16_bits(a) for a in I.generate(T, D, F, seed=T))
    ws = gmlp.Workspace(T, D, F)
    want_y = gmlp.forward(x, wg, wu, wd, path=path, workspace=ws, rmsnorm=True)
    want_h = gmlp.gate_up(x, wg, wu, path=path, workspace=ws)
    want_d = gmlp.down(want_h, wd, path=path, workspace=ws)
    n = gmlp.workspace_size(T, D, F)
    code = gmlp._PATHS[path] | FRESH
    for _ in range(2):
        y, h, d = torch.empty_like(want_y), torch.empty_like(want_h), torch.empty_like(want_d)
        t, p = _dirty(n)
        assert lib.gmlp_forward_variant(x.data_ptr(), wg.data_ptr(), wu.data_ptr(), wd.data_ptr(), y.data_ptr(), T, D,
                                        F, 0, 1.0, 1, 1e-6, code, p, n, gmlp._stream(None)) == 0
        t.fill_(0xFF)
        assert lib.gmlp_gate_up_ws(x.data_ptr(), wg.data_ptr(), wu.data_ptr(), h.data_ptr(), T, D, F, code, p, n,
                                   gmlp._stream(None)) == 0
        t.fill_(0xFF)
        assert lib.gmlp_down_ws(want_h.data_ptr(), wd.data_ptr(), d.data_ptr(), T, F, D, code, p, n,
                                gmlp._stream(None)) == 0
        for got, want in ((y, want_y), (h, want_h), (d, want_d)):
            assert torch.equal(got.view(torch.int16), want.view(torch.int16))
    # The binding without a workspace, and the C entry point that allocates.
    assert torch.equal(gmlp.forward(x, wg, wu, wd, path=path, rmsnorm=True).view(torch.int16), want_y.view(torch.int16))
    if path == "auto":
        plain = gmlp.forward(x, wg, wu, wd, workspace=ws)
        y = torch.empty_like(plain)
        assert lib.gmlp_forward(x.data_ptr(), wg.data_ptr(), wu.data_ptr(), wd.data_ptr(), y.data_ptr(), T, D, F,
                                gmlp._stream(None)) == 0
        assert torch.equal(y.view(torch.int16), plain.view(torch.int16))


@pytest.mark.gpu
@pytest.mark.parametrize("M,K,N", [(3, 520, 264), (100, 2056, 1544), (300, 4104, 2056), (9, 72, 16384)])
def test_fresh_softmax_matmul(M, K, N):
    lib = gmlp.library()
    X, Y = I.generate_softmax_matmul(M, K, N, seed=M)
    x, y = gmlp.from_bf16_bits(X), gmlp.from_bf16_bits(Y)
    want = smm.softmax_matmul(x, y, workspace=smm.make_workspace(M, K, N))
    n = smm.workspace_size(M, K, N)
    for _ in range(2):
        z = torch.empty_like(want)
        t, p = _dirty(n)
        assert lib.softmax_matmul_ws(x.data_ptr(), y.data_ptr(), z.data_ptr(), M, K, N, FRESH, p, n,
                                     gmlp._stream(None)) == 0
        assert torch.equal(z.view(torch.int16), want.view(torch.int16))
    assert torch.equal(smm.softmax_matmul(x, y).view(torch.int16), want.view(torch.int16))


@pytest.mark.gpu
def test_calls_without_a_workspace_are_captured():
    x, wg, wu, wd = (gmlp.from_bf16_bits(a) for a in I.generate(100, 2056, 1544, seed=1))
    xs, ys = (gmlp.from_bf16_bits(a) for a in I.generate_softmax_matmul(64, 2056, 1032, seed=2))
    side = torch.cuda.Stream()
    with torch.cuda.stream(side):
        gmlp.forward(x, wg, wu, wd), smm.softmax_matmul(xs, ys)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        y = gmlp.forward(x, wg, wu, wd)
        z = smm.softmax_matmul(xs, ys)
    for i in range(4):
        x.mul_(-1 if i % 2 else 1)
        y.zero_(), z.zero_()
        g.replay()
        want_y, want_z = gmlp.forward(x, wg, wu, wd), smm.softmax_matmul(xs, ys)
        torch.cuda.synchronize()
        assert np.array_equal(gmlp.to_bf16_bits(y), gmlp.to_bf16_bits(want_y))
        assert np.array_equal(gmlp.to_bf16_bits(z), gmlp.to_bf16_bits(want_z))


@pytest.mark.gpu
def test_a_stream_known_by_its_handle_only():
    # All that a call asks of a stream is its cuda_stream, also where it takes
    # scratch memory (which it takes on that stream).
    class Handle:
        def __init__(self, stream):
            self.cuda_stream = stream.cuda_stream

    side = torch.cuda.Stream()
    x, wg, wu, wd = (gmlp.from_bf16_bits(a) for a in I.generate(100, 2056, 1544, seed=1))
    want = gmlp.forward(x, wg, wu, wd)
    torch.cuda.synchronize()
    before = torch.cuda.current_stream()
    y, h, d = torch.empty_like(want), torch.empty(100, 1544, dtype=torch.bfloat16, device="cuda"), torch.empty_like(want)
    gmlp.forward(x, wg, wu, wd, out=y, stream=Handle(side))
    gmlp.gate_up(x, wg, wu, out=h, stream=Handle(side))
    gmlp.down(h, wd, out=d, stream=Handle(side))
    z = smm.softmax_matmul(x, wg, stream=Handle(side))
    torch.cuda.synchronize()
    assert torch.cuda.current_stream() == before
    for got in (y, d):
        assert torch.equal(got.view(torch.int16), want.view(torch.int16))
    assert torch.equal(z.view(torch.int16), smm.softmax_matmul(x, wg).view(torch.int16))


def test_a_refused_shape_is_reported_as_before():
    # No device needed: the shape is refused before anything is allocated.
    assert gmlp._scratch(0, 4, "cuda", None, True, "unused") == (None, None)
    assert gmlp._scratch(1024, 0, "cuda", None, True, "unused") == (None, None)
    with pytest.raises(ValueError, match="invalid shape"):
        gmlp._scratch(0, 4, "cuda", None, False, "invalid shape T=4 D=12 F=16")


def test_scratch_is_memory_of_the_device_of_the_stream(monkeypatch):
    # The arguments on another device than the current one, whose stream the
    # calls run on: the outputs are allocated on the arguments' device, the
    # scratch on "cuda", the device of the stream.
    class Library:
        def __getattr__(self, name):
            return lambda *args: 4096 if name.endswith("workspace_size") else 0

    asked = []

    def empty(shape, dtype, device, stream=None):
        asked.append((dtype, str(device), stream))
        return torch.empty(shape, dtype=dtype)

    for module in (gmlp, smm):
        monkeypatch.setattr(module, "library", Library)
        monkeypatch.setattr(module, "_empty", empty)
        monkeypatch.setattr(module, "_expect", lambda *args: None)
        monkeypatch.setattr(module, "_stream", lambda stream: 0)
    a = torch.empty(16, 16, dtype=torch.bfloat16)
    for call in (lambda s: gmlp.forward(a, a, a, a, stream=s), lambda s: gmlp.gate_up(a, a, a, stream=s),
                 lambda s: gmlp.down(a, a, stream=s), lambda s: smm.softmax_matmul(a, a, stream=s),
                 lambda s: gmlp.forward(a, a, a, a, stream=s, path="mfma", rmsnorm=True)):
        for stream in (None, "a stream"):
            asked.clear()
            call(stream)
            assert asked == [(torch.bfloat16, "cpu", stream), (torch.uint8, "cuda", stream)]
