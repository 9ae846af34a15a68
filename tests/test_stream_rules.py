"""Where the automatic path takes the streaming tiles and how it splits K for
them (on the CPU), and the kernels on either side of each line against the
oracle (on the GPU)."""
import numpy as np
import pytest
import torch

import oracle
from paper_2606_26344_amd import gmlp
from paper_2606_26344_amd import inputs as I
from paper_2606_26344_amd import softmax_matmul as smm

from test_gpu_parity import _check


def _stream(line):
    return ", 128>" in line[0]


# Gate/up, 64-column tiles: each range of K from 513 to 1408 rows with as many
# output columns as it takes shorter splits for, and with more; other lengths
# in splits of 512 rows and more.
SPLITS = [(97, 584, 1024, 2), (97, 584, 1032, 1), (97, 584, 128, 1), (96, 584, 264, 1),
          (31, 640, 264, 1), (31, 648, 5440, 3), (31, 648, 5448, 1), (97, 768, 2688, 3), (97, 768, 2696, 1),
          (97, 776, 4096, 3), (97, 776, 4104, 1), (96, 896, 5440, 3),
          (64, 1024, 2048, 4), (64, 1024, 2056, 2), (64, 1024, 4096, 2), (97, 904, 1024, 4), (97, 904, 1032, 2),
          (64, 1032, 264, 3), (97, 1280, 2688, 3), (97, 1280, 2696, 2), (97, 1288, 4096, 3), (97, 1288, 4104, 2),
          (96, 1032, 5440, 3), (113, 1336, 272, 3), (29, 1296, 856, 3), (40, 1416, 264, 3), (69, 6888, 544, 11)]


@pytest.mark.parametrize("T,D,F,splits", SPLITS)
def test_gate_up_splits(T, D, F, splits):
    line = gmlp.describe(T, D, F)[0]
    assert _stream(line) and line[3] == splits, line
    assert line[1] == -(-F // 64) * splits


# (T, columns, K, streaming): both sides of each line of the rule.
GATE_UP = [(81, 1000, 64, False), (81, 1000, 72, True), (80, 1000, 64, True), (96, 80, 64, False),
           (97, 80, 192, False), (97, 1000, 200, True), (128, 3144, 8, False), (128, 3144, 192, False),
           (128, 128, 568, True), (128, 136, 568, False), (113, 2752, 520, False), (113, 2760, 520, True),
           (112, 1600, 576, False), (112, 1608, 576, True), (97, 264, 512, True), (97, 264, 584, True), (96, 264, 520, True),
           (20, 8200, 1104, False), (20, 8200, 1096, True), (120, 8704, 1920, False), (48, 8704, 1296, True),
           (48, 8704, 1304, False), (97, 9608, 1200, True), (97, 9608, 1208, False), (96, 9608, 1400, True),
           (96, 9608, 1408, False), (120, 8192, 2048, True)]
DOWN = [(48, 9216, 1280, True), (48, 9216, 1288, False), (96, 9608, 1504, True), (96, 9608, 1512, False),
        (97, 9608, 1280, True), (97, 9608, 1288, False), (64, 16384, 1016, True), (64, 16392, 192, True),
        (64, 16392, 200, False), (65, 16392, 16, False), (80, 32776, 16, True), (81, 32776, 16, False),
        (120, 8, 192, True), (128, 8192, 2048, True)]


@pytest.mark.parametrize("T,F,D,stream", GATE_UP)
def test_gate_up_tile(T, F, D, stream):
    assert _stream(gmlp.describe(T, D, F)[0]) == stream


@pytest.mark.parametrize("T,D,F,stream", DOWN)
def test_down_tile(T, D, F, stream):
    assert _stream(gmlp.describe(T, D, F)[1]) == stream


@pytest.mark.gpu
@pytest.mark.parametrize("T,D,F,splits", SPLITS)
def test_gate_up_split_kernels(orc, T, D, F, splits):
    X, Wg, Wu, Wd = I.generate(T, D, F, seed=T + D)
    ws = gmlp.Workspace(T, D, F)
    h = [gmlp.gate_up(*(gmlp.from_bf16_bits(a) for a in (X, Wg, Wu)), workspace=ws) for _ in range(2)]
    torch.cuda.synchronize()
    assert torch.equal(h[0].view(torch.int16), h[1].view(torch.int16))
    _, ref = orc.gated_mlp_rows(X, Wg, Wu, Wd, return_h=True)
    _check(gmlp.to_bf16_bits(h[0]), ref, "T=%d D=%d F=%d" % (T, D, F))


# The steps that went back to the ring, one of each kind, with the options.
@pytest.mark.gpu
@pytest.mark.parametrize("T,D,F", [(96, 64, 1000), (128, 8, 3144), (100, 568, 1544), (97, 192, 80), (120, 1912, 8712), (20, 1104, 8200)])
def test_gate_up_on_the_ring(orc, T, D, F):
    assert not _stream(gmlp.describe(T, D, F)[0])
    variant = dict(activation="swish", beta=1.702, rmsnorm=True, eps=1e-5)
    X, Wg, Wu, Wd = I.generate(T, D, F, seed=T + D)
    h = gmlp.gate_up(*(gmlp.from_bf16_bits(a) for a in (X, Wg, Wu)), workspace=gmlp.Workspace(T, D, F), **variant)
    torch.cuda.synchronize()
    rows = np.unique(np.concatenate([I.sample_rows(T, 12), np.arange(T - 2, T)]))
    _, ref = orc.gated_mlp_rows(X, Wg, Wu, Wd, rows=rows, return_h=True, **variant)
    _check(gmlp.to_bf16_bits(h)[rows], ref, "T=%d D=%d F=%d" % (T, D, F))


@pytest.mark.gpu
@pytest.mark.parametrize("M,K,N", [(48, 1288, 9216), (65, 16, 16392), (64, 200, 16392), (81, 72, 32776)])
def test_softmax_matmul_on_the_ring(M, K, N):
    assert not _stream(smm.describe(M, K, N)[1])
    X, Y = I.generate_softmax_matmul(M, K, N, seed=M)
    z = smm.softmax_matmul(gmlp.from_bf16_bits(X), gmlp.from_bf16_bits(Y), workspace=smm.make_workspace(M, K, N))
    torch.cuda.synchronize()
    _check(gmlp.to_bf16_bits(z), oracle.softmax_matmul_rows(X, Y),
           "M=%d K=%d N=%d" % (M, K, N))
