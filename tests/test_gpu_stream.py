"""The streaming MFMA kernels (6 to 128 tokens, small weights) against the
oracle and against the LDS-ring kernels of the explicit "mfma" path, at the
edges of their tiles: 16-token tiles (15 .. 17, ... 112, 113, 128 tokens), 64-
and 128-column tiles cut short by F or D, K tails shorter than a 32-row batch,
one split and many, waves without a batch (K = 8), and every epilogue.

Both paths add the same bf16 products in fp32, in another order, and round
once: an element differs by at most one bf16 step (2^-8 of its value) plus,
after the down step, what single-step differences of H give (2^-8 of H's rms
over many terms); the oracle's rule |got - ref| <= 1e-2 (|ref| + rms) covers
both, and is asserted for either reference.
"""
import numpy as np
import pytest
import torch

import oracle
from paper_2606_26344_amd import gmlp
from paper_2606_26344_amd import inputs as I
from paper_2606_26344_amd import softmax_matmul as smm

pytestmark = pytest.mark.gpu

TOL = 1e-2


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    assert torch.cuda.is_available(), "GPU tests need a HIP device"
    gmlp.library()


def _f64(t):
    return I.bf16_bits_to_f32(gmlp.to_bf16_bits(t)).astype(np.float64)


def _check(got, ref, what):
    assert np.all(np.isfinite(got)), what
    bound = TOL * (np.abs(ref) + np.sqrt(np.mean(ref ** 2)))
    ratio = float(np.max(np.abs(got - ref) / bound))
    print("%s max err/bound = %.3f" % (what, ratio), flush=True)
    assert ratio <= 1.0, what


def _is_stream(line):
    return line[0].startswith("gemm_mfma_kernel<GemmShape<") and ", 128>" in line[0]


# T, D, F: 64-column tiles in both steps unless noted.
SHAPES = [(T, 264, 520) for T in (6, 15, 16, 17, 31, 32, 33, 48, 49, 64, 65, 80, 81, 96, 97, 112, 113, 128)]
SHAPES += [(24, 8, 8), (7, 8, 1032), (40, 1032, 8), (80, 40, 72), (128, 40, 72),   # waves without a batch, one short tile
           (16, 2056, 3080), (9, 1032, 4104), (16, 3080, 2056),      # 128-column tiles (weights above 2^22), short last tile
           (51, 1032, 4104), (100, 2056, 1544), (128, 1544, 4168),    # several splits, ragged K
           (64, 4104, 264), (90, 136, 11000)]


@pytest.mark.parametrize("T,D,F", SHAPES, ids=["T%dD%dF%d" % s for s in SHAPES])
def test_stream_tiles(orc, T, D, F):
    plan = gmlp.describe(T, D, F)
    # (128 tokens over 40 rows: the gate/up step runs on the ring, which is faster there.)
    assert [_is_stream(line) for line in plan] == [(T, D) != (128, 40), True], plan
    X, Wg, Wu, Wd = I.generate(T, D, F, seed=T + D + F)
    x, wg, wu, wd = (gmlp.from_bf16_bits(a) for a in (X, Wg, Wu, Wd))
    ws = gmlp.Workspace(T, D, F)
    h = gmlp.gate_up(x, wg, wu, workspace=ws)
    y = gmlp.down(h, wd, workspace=ws)
    y2 = gmlp.forward(x, wg, wu, wd, workspace=ws)
    ring_h = gmlp.gate_up(x, wg, wu, path="mfma", workspace=ws)
    ring_y = gmlp.down(h, wd, path="mfma", workspace=ws)
    again = gmlp.forward(x, wg, wu, wd, workspace=ws)
    torch.cuda.synchronize()
    assert torch.equal(y.view(torch.int16), y2.view(torch.int16))
    assert torch.equal(again.view(torch.int16), y2.view(torch.int16))
    assert int(torch.count_nonzero(ws.buffer[:128 * 1024])) == 0  # counters back at zero
    rows = np.arange(T) if T * D * F < 2 ** 27 else I.sample_rows(T, 24)
    _, H_ref = orc.gated_mlp_rows(X, Wg, Wu, Wd, rows=rows, return_h=True)
    what = "T=%d D=%d F=%d" % (T, D, F)
    _check(_f64(h)[rows], H_ref, "H " + what)
    _check(_f64(y)[rows], orc.down_rows(gmlp.to_bf16_bits(h)[rows], Wd), "Y " + what)
    _check(_f64(h), _f64(ring_h), "H against the ring " + what)
    _check(_f64(y), _f64(ring_y), "Y against the ring " + what)


@pytest.mark.parametrize("T", [16, 40, 90, 128])
@pytest.mark.parametrize("variant", [dict(rmsnorm=True, eps=1e-5), dict(activation="swish", beta=1.702, rmsnorm=True),
                                     dict(activation="sigmoid")], ids=["rmsnorm", "rmsnorm_swiglu", "glu"])
def test_stream_variants(orc, T, variant):
    D, F = 520, 1032
    X, Wg, Wu, Wd = I.generate(T, D, F, seed=T)
    args = [gmlp.from_bf16_bits(a) for a in (X, Wg, Wu, Wd)]
    # (128 tokens over 520 rows: the gate/up step runs on the ring, which is faster there.)
    assert [_is_stream(line) for line in gmlp.describe(T, D, F)] == [T != 128, True]
    y = gmlp.forward(*args, workspace=gmlp.Workspace(T, D, F), **variant)
    torch.cuda.synchronize()
    _check(_f64(y), orc.gated_mlp_rows(X, Wg, Wu, Wd, **variant), "T=%d %s" % (T, variant))


# The options where test_stream_variants does not reach: the 128-column gate/up
# tile (up to 16 tokens, weights above 2^22), and the epilogue after the split-K
# exchange of every tile.
@pytest.mark.parametrize("T,D,F,columns,splits", [(16, 2056, 3080, 128, 6), (9, 1032, 4104, 128, 3), (30, 1288, 1544, 64, 3),
                                                  (60, 1032, 2056, 64, 3), (90, 2056, 1544, 64, 4),
                                                  (100, 2056, 1544, 64, 4), (128, 1544, 4168, 64, 3)])
@pytest.mark.parametrize("variant", [dict(rmsnorm=True, eps=1e-5), dict(activation="swish", beta=1.702, rmsnorm=True),
                                     dict(activation="sigmoid")], ids=["rmsnorm", "rmsnorm_swiglu", "glu"])
def test_stream_variants_after_the_exchange(orc, T, D, F, columns, splits, variant):
    name, grid, _, got = gmlp.describe(T, D, F)[0]
    tile = "GemmShape<2, 4, 1, 1, 1, 1, 128>" if columns == 128 else "GemmShape<2, 2, 1, 1, %d, 2, 128>" % -(-T // 32)
    assert tile in name and got == splits and grid == -(-F // columns) * splits, (name, grid, got)
    X, Wg, Wu, Wd = I.generate(T, D, F, seed=T + F)
    h = gmlp.gate_up(*(gmlp.from_bf16_bits(a) for a in (X, Wg, Wu)), workspace=gmlp.Workspace(T, D, F), **variant)
    torch.cuda.synchronize()
    rows = np.arange(T) if T <= 16 else np.unique(np.concatenate([I.sample_rows(T, 24), np.arange(T - 2, T)]))
    _, ref = orc.gated_mlp_rows(X, Wg, Wu, Wd, rows=rows, return_h=True, **variant)
    _check(_f64(h)[rows], ref, "T=%d D=%d F=%d %s" % (T, D, F, variant))


# The streaming tiles as the rest of a token split of the gate/up step: their
# rows start past the whole tiles' in X, H and the row scales.
@pytest.mark.parametrize("T,D,F", [(560, 1032, 12288), (530, 264, 12280), (1600, 2048, 8192)])
def test_stream_rest_of_a_token_split(orc, T, D, F):
    plan = gmlp.describe(T, D, F)
    assert len(plan) == 3 and _is_stream(plan[1]) and ", 0, true, true>" in plan[1][0], plan
    variant = dict(activation="swish", beta=1.702, rmsnorm=True, eps=1e-5)
    X, Wg, Wu, Wd = I.generate(T, D, F, seed=T + F)
    x, wg, wu, wd = (gmlp.from_bf16_bits(a) for a in (X, Wg, Wu, Wd))
    ws = gmlp.Workspace(T, D, F)
    h = torch.full((T, F), float("nan"), dtype=torch.bfloat16, device="cuda")
    gmlp.gate_up(x, wg, wu, out=h, workspace=ws, **variant)
    y = gmlp.forward(x, wg, wu, wd, workspace=ws, **variant)
    torch.cuda.synchronize()
    assert bool(torch.isfinite(h).all())  # every element written
    first = T // 256 * 256
    rows = np.unique(np.concatenate([I.sample_rows(T, 8), np.arange(first - 2, first + 6), np.arange(T - 4, T)]))
    Y_ref, H_ref = orc.gated_mlp_rows(X, Wg, Wu, Wd, rows=rows, return_h=True, **variant)
    _check(_f64(h)[rows], H_ref, "H T=%d D=%d F=%d" % (T, D, F))
    _check(_f64(y)[rows], Y_ref, "Y T=%d D=%d F=%d" % (T, D, F))


@pytest.mark.parametrize("M,K,N", [(9, 520, 264), (33, 1032, 72), (100, 2056, 1032), (16, 4104, 1544), (128, 72, 520)])
def test_stream_softmax_matmul(M, K, N):
    assert _is_stream(smm.describe(M, K, N)[1])
    X, Y = I.generate_softmax_matmul(M, K, N, seed=M)
    z = smm.softmax_matmul(gmlp.from_bf16_bits(X), gmlp.from_bf16_bits(Y), workspace=smm.make_workspace(M, K, N))
    torch.cuda.synchronize()
    _check(_f64(z), oracle.softmax_matmul_rows(X, Y), "M=%d K=%d N=%d" % (M, K, N))


# The last block of a tile adds the other splits in groups (32, 8 and 2 of
# them for one token tile of a down step, fewer for more): two splits to some
# sixty, whole groups and every kind of remainder, with one, two, four and
# eight 16-token tiles.
@pytest.mark.parametrize("K", [1032, 1544, 2056, 3080, 5128, 9224, 17416, 33800])
@pytest.mark.parametrize("T", [8, 24, 64, 128])
def test_stream_split_exchange(orc, T, K):
    N = 72
    down, gate_up = gmlp.describe(T, N, K)[1], gmlp.describe(T, K, N)[0]
    assert _is_stream(down) and _is_stream(gate_up) and down[3] > 1 and gate_up[3] > 1, (down, gate_up)
    print("T=%d K=%d splits: down %d, gate/up %d" % (T, K, down[3], gate_up[3]), flush=True)
    ws, ws2 = gmlp.Workspace(T, N, K), gmlp.Workspace(T, K, N)
    rng = np.random.default_rng(T + K)
    H, Wd = (I.f32_to_bf16_bits(rng.standard_normal(s).astype(np.float32) * a)
             for s, a in (((T, K), 1.0), ((K, N), K ** -0.5)))
    y = [gmlp.down(gmlp.from_bf16_bits(H), gmlp.from_bf16_bits(Wd), workspace=ws) for _ in range(2)]
    _check(_f64(y[0]), orc.down_rows(H, Wd), "down T=%d K=%d" % (T, K))
    X, Wg, Wu, Wd = I.generate(T, K, N, seed=T + K)
    h = [gmlp.gate_up(*(gmlp.from_bf16_bits(a) for a in (X, Wg, Wu)), workspace=ws2) for _ in range(2)]
    _, ref = orc.gated_mlp_rows(X, Wg, Wu, Wd, return_h=True)
    _check(_f64(h[0]), ref, "H T=%d K=%d" % (T, K))
    for w, (a, b) in ((ws, y), (ws2, h)):
        assert torch.equal(a.view(torch.int16), b.view(torch.int16))
        assert int(torch.count_nonzero(w.buffer[:128 * 1024])) == 0  # counters back at zero


@pytest.mark.parametrize("T", [16, 70])
def test_stream_specials(T):
    # A row with a NaN, a weight column with an infinity: each stays in its
    # row and its column, also past the K tail and the token tail, where the
    # kernel multiplies zeros.
    D, F = 1032, 520
    X, Wg, Wu, Wd = I.generate(T, D, F, seed=3)
    Wd = Wd.copy()
    H = I.f32_to_bf16_bits(np.abs(np.random.default_rng(1).standard_normal((T, F))).astype(np.float32) + 0.5)
    Wd[F - 1, 5] = 0x7F80  # +inf
    H[T - 1, F - 3] = 0x7FC0  # NaN
    y = I.bf16_bits_to_f32(gmlp.to_bf16_bits(gmlp.down(gmlp.from_bf16_bits(H), gmlp.from_bf16_bits(Wd))))
    assert np.all(np.isnan(y[T - 1]))
    assert np.all(np.isposinf(y[:T - 1, 5]))
    assert np.all(np.isfinite(np.delete(y[:T - 1], 5, axis=1)))
