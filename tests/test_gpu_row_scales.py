"""The row scales of RMSNorm on the MFMA path: rows of one 16-byte chunk, rows
that fill one pass of the kernel's block and rows past it (D > 8192), against
the oracle."""
import numpy as np
import pytest
import torch

from paper_2606_26344_amd import gmlp
from paper_2606_26344_amd import inputs as I

TOL = 1e-2


def _check(got, ref, what):
    assert np.all(np.isfinite(got)), what
    ratio = float(np.max(np.abs(got - ref) / (TOL * (np.abs(ref) + np.sqrt(np.mean(ref ** 2))))))
    print("%s max err/bound = %.3f" % (what, ratio), flush=True)
    assert ratio <= 1.0, what


@pytest.mark.gpu
@pytest.mark.parametrize("T,D", [(6, 8), (7, 72), (130, 2040), (9, 2056), (20, 8192), (13, 8200), (6, 16392)])
def test_row_scales(orc, T, D):
    F = 72
    X, Wg, Wu, Wd = I.generate(T, D, F, seed=D)
    variant = dict(rmsnorm=True, eps=1e-5)
    h = gmlp.gate_up(*(gmlp.from_bf16_bits(a) for a in (X, Wg, Wu)), **variant)
    torch.cuda.synchronize()
    _, ref = orc.gated_mlp_rows(X, Wg, Wu, Wd, return_h=True, **variant)
    _check(I.bf16_bits_to_f32(gmlp.to_bf16_bits(h)).astype(np.float64), ref, "T=%d D=%d" % (T, D))
