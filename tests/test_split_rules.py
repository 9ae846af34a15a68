"""How K is split above 128 tokens: few splits where K is short, since the
last block of a tile reads every split's fp32 partial tile.  The plans on the
CPU; the kernels at those splits on the GPU, against the oracle."""
import numpy as np
import pytest
import torch

from paper_2606_26344_amd import gmlp
from paper_2606_26344_amd import inputs as I

TOL = 1e-2


@pytest.mark.parametrize("T,D,F,gu,dn", [(3982, 256, 512, 1, 1), (211, 1032, 2056, 1, 3), (222, 4096, 16384, 1, 4),
                                         (330, 1648, 4848, 2, 6)])
def test_splits(T, D, F, gu, dn):
    plan = gmlp.describe(T, D, F)
    assert [line[3] for line in plan] == [gu, dn], plan


@pytest.mark.parametrize("T", [129, 160, 192, 193, 256, 300, 500, 1000])
@pytest.mark.parametrize("D,F", [(8, 8), (72, 2056), (264, 520), (1032, 4104), (2048, 8192), (4096, 14336)])
def test_splits_fit_a_round(T, D, F):
    # (None of these plans has split tail tiles.)
    for (name, grid, _, splits), M, K in zip(gmlp.describe(T, D, F), (F, D), (D, F)):
        wm, wn, tm, tn, _, bk = [int(v) for v in name.split("GemmShape<")[1].split(">")[0].split(",")][1:7]
        tiles = -(-M // (32 * wm * tm)) * -(-T // (32 * wn * tn))
        pair = name.endswith(", 2, true, true>")  # a G and a U block per tile, each over all of K
        assert grid == tiles * splits, (name, grid, splits)
        assert splits == 1 or grid <= 256, (name, grid, splits)
        assert splits == 2 if pair else 1 <= splits <= max(1, -(-K // bk) // 2), (name, splits)


# Down steps of 257 to 384 tokens and 64 to 128 192-token tiles: where K is
# short the steps are hardly split, and unsplit 192-token tiles are longer blocks
# on fewer CUs than the 128-token ones.
SHORT_K = [(300, 4096, 1024), (300, 6144, 1024), (384, 4096, 1032), (300, 4096, 512), (257, 8192, 768)]
LONG_K = [(257, 4096, 14336), (300, 4096, 4096), (384, 4096, 14336), (320, 8192, 28672)]


@pytest.mark.parametrize("T,D,F", SHORT_K + LONG_K)
def test_down_tile_of_257_to_384_tokens(T, D, F):
    name, grid, _, splits = gmlp.describe(T, D, F)[-1]
    tokens = 128 if (T, D, F) in SHORT_K else 192
    tile = {128: "GemmShape<1, 2, 2, 2, 2, 4, 64>", 192: "GemmShape<1, 4, 1, 1, 6, 3, 64>"}[tokens]
    assert tile in name and grid == -(-T // tokens) * -(-D // 128) * splits, (name, grid, splits)
    assert splits > 1 or tokens == 128


def _check(got, ref, what):
    assert np.all(np.isfinite(got)), what
    ratio = float(np.max(np.abs(got - ref) / (TOL * (np.abs(ref) + np.sqrt(np.mean(ref ** 2))))))
    print("%s max err/bound = %.3f" % (what, ratio), flush=True)
    assert ratio <= 1.0, what


@pytest.mark.gpu
@pytest.mark.parametrize("T,D,F", [(390, 256, 512), (211, 1032, 2056), (140, 1032, 4104), (170, 520, 1544),
                                   (330, 1032, 4848), (768, 2760, 1544), (300, 4096, 520)])
def test_split_kernels(orc, T, D, F):
    X, Wg, Wu, Wd = I.generate(T, D, F, seed=T)
    x, wg, wu, wd = (gmlp.from_bf16_bits(a) for a in (X, Wg, Wu, Wd))
    ws = gmlp.Workspace(T, D, F)
    y = gmlp.forward(x, wg, wu, wd, workspace=ws)
    again = gmlp.forward(x, wg, wu, wd, workspace=ws)
    torch.cuda.synchronize()
    assert torch.equal(y.view(torch.int16), again.view(torch.int16))
    rows = np.unique(np.concatenate([I.sample_rows(T, 24), np.arange(T - 4, T)]))
    _check(I.bf16_bits_to_f32(gmlp.to_bf16_bits(y)[rows]).astype(np.float64),
           orc.gated_mlp_rows(X, Wg, Wu, Wd, rows=rows), "T=%d D=%d F=%d" % (T, D, F))
