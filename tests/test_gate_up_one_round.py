"""Gate/up at 129 to 256 tokens with more than 128 column tiles: one 192- or
256-token tile per column tile, weights streamed, in a single round of blocks
(two 128-token tiles of each would take a second one)."""
import numpy as np
import pytest
import torch

from paper_2606_26344_amd import gmlp
from paper_2606_26344_amd import inputs as I

TOL = 1e-2


@pytest.mark.parametrize("F,one", [(16384, False), (16392, True), (24576, True), (32768, True), (32776, False)])
@pytest.mark.parametrize("T", [128, 129, 192, 193, 256, 257])
def test_plan(T, F, one):
    name, grid, _, splits = gmlp.describe(T, 520, F)[0]
    tile = "GemmShape<2, 4, 1, 1, 6, 4, 32>, 0, false, true>" if T <= 192 else "GemmShape<2, 4, 2, 1, 4, 2, 64>, 0, false, true>"
    assert (tile in name) == (one and 128 < T <= 256), name
    if one and 128 < T <= 256:
        assert grid == -(-F // 128) and splits == 1


@pytest.mark.gpu
@pytest.mark.parametrize("T,D,F", [(129, 72, 16392), (192, 520, 17000), (193, 264, 32768), (250, 520, 16648), (256, 136, 20488)])
def test_against_the_oracle(orc, T, D, F):
    X, Wg, Wu, Wd = I.generate(T, D, F, seed=T)
    x, wg, wu = (gmlp.from_bf16_bits(a) for a in (X, Wg, Wu))
    h = torch.full((T, F), float("nan"), dtype=torch.bfloat16, device="cuda")
    gmlp.gate_up(x, wg, wu, out=h, workspace=gmlp.Workspace(T, D, F), activation="swish", beta=1.702, rmsnorm=True)
    torch.cuda.synchronize()
    got = I.bf16_bits_to_f32(gmlp.to_bf16_bits(h)).astype(np.float64)
    assert np.all(np.isfinite(got))  # every element written
    rows = np.unique(np.concatenate([I.sample_rows(T, 8), np.arange(T - 3, T)]))
    _, ref = orc.gated_mlp_rows(X, Wg, Wu, Wd, rows=rows, return_h=True, activation="swish", beta=1.702, rmsnorm=True)
    ratio = float(np.max(np.abs(got[rows] - ref) / (TOL * (np.abs(ref) + np.sqrt(np.mean(ref ** 2))))))
    print("T=%d D=%d F=%d max err/bound = %.3f" % (T, D, F, ratio), flush=True)
    assert ratio <= 1.0
