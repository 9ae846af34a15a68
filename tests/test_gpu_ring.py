"""The LDS-ring tiles at 6 to 128 tokens against the oracle, on the explicit
"mfma" path: the automatic path runs the streaming tiles for most weights
that a test can afford, and takes the ring for large weights and for the steps
that are faster on it.  Every tile (32, 64, 96 and 128 tokens) at its edges, with
and without splits of K, and every epilogue: SiLU, SwiGLU behind RMSNorm, GLU, and the
row divisors of Softmax+MatMul.  The tiles are asserted by name."""
import numpy as np
import pytest
import torch

import oracle
from paper_2606_26344_amd import gmlp
from paper_2606_26344_amd import inputs as I
from paper_2606_26344_amd import softmax_matmul as smm

from test_gpu_parity import _check, _dev

pytestmark = pytest.mark.gpu

VARIANTS = {"silu": {}, "rmsnorm_swiglu": dict(activation="swish", beta=1.702, rmsnorm=True, eps=1e-5),
            "glu": dict(activation="sigmoid")}
# Tokens -> (gate/up, down) tile.
TILES = {32: ("GemmShape<2, 4, 1, 1, 1, 4, 64>", "GemmShape<1, 4, 1, 1, 1, 6, 64>"),
         64: ("GemmShape<2, 4, 1, 1, 2, 3, 64>", "GemmShape<1, 4, 1, 1, 2, 6, 64>"),
         96: ("GemmShape<2, 4, 1, 1, 3, 3, 64>", "GemmShape<1, 4, 1, 1, 3, 5, 64>"),
         128: ("GemmShape<2, 4, 2, 1, 2, 3, 64>", "GemmShape<1, 2, 2, 2, 2, 4, 64>")}


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    assert torch.cuda.is_available(), "GPU tests need a HIP device"
    gmlp.library()


def _tiles(T):
    return TILES[min(t for t in TILES if T <= t)]


@pytest.mark.parametrize("variant", sorted(VARIANTS))
@pytest.mark.parametrize("D,F", [(72, 136), (1032, 520), (520, 2056)])
@pytest.mark.parametrize("T", [6, 17, 32, 33, 64, 65, 96, 97, 128])
def test_ring_tiles(orc, T, D, F, variant):
    plan = gmlp.describe(T, D, F, path="mfma")
    for line, tile, K in zip(plan, _tiles(T), (D, F)):
        assert tile in line[0] and (line[3] > 1) == (K > 192), plan
    X, Wg, Wu, Wd = I.generate(T, D, F, seed=T + D)
    x, wg, wu, wd = (_dev(a) for a in (X, Wg, Wu, Wd))
    ws = gmlp.Workspace(T, D, F)
    h = gmlp.gate_up(x, wg, wu, path="mfma", workspace=ws, **VARIANTS[variant])
    y = gmlp.down(h, wd, path="mfma", workspace=ws)
    torch.cuda.synchronize()
    _, ref = orc.gated_mlp_rows(X, Wg, Wu, Wd, return_h=True, **VARIANTS[variant])
    what = "T=%d D=%d F=%d %s" % (T, D, F, variant)
    _check(gmlp.to_bf16_bits(h), ref, "H " + what)
    _check(gmlp.to_bf16_bits(y), orc.down_rows(gmlp.to_bf16_bits(h), Wd), "Y " + what)


@pytest.mark.parametrize("K,N", [(136, 264), (1032, 520), (4104, 136)])
@pytest.mark.parametrize("M", [9, 16, 33, 64, 80, 96, 100, 127, 128])
def test_ring_softmax_matmul(M, K, N):
    line = smm.describe(M, K, N, path="mfma")[1]
    assert _tiles(M)[1] in line[0] and (line[3] > 1) == (K > 192), line
    X, Y = I.generate_softmax_matmul(M, K, N, seed=M + K)
    z = smm.softmax_matmul(_dev(X), _dev(Y), path="mfma", workspace=smm.make_workspace(M, K, N))
    torch.cuda.synchronize()
    _check(gmlp.to_bf16_bits(z), oracle.softmax_matmul_rows(X, Y), "M=%d K=%d N=%d" % (M, K, N))
