"""GPU parity of the float32 cross-Gram's split-product tiles (factorized route)
against the float64 oracle where they can go wrong: 128-row token tiles that
lie wholly past their examples' lengths, halves of a tile past them, feature
widths ending inside a 32-feature stage, and values the three-term bf16 split
cannot carry.  Bounds as in test_gpu_crossgram.py (1e-5 relative Frobenius
error, float32 products and sums of exact inputs)."""
import numpy as np
import pytest
import torch

import paper_2609_38767_amd as dt
from gpu_util import host64, rel_fro
from oracle import crossgram as ocg
from paper_2609_38767_amd.session import cross_gram, sq_norms
from test_gpu_crossgram import _batch, _oracle_batch, _session

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("dims", [[(72, 200)], [(36, 8), (4, 260), (128, 32)]])
def test_cross_gram_dead_tiles(dtype, dims):
    dims = [(8 * ((a + 7) // 8), 8 * ((b + 7) // 8)) for a, b in dims] if dtype == "bf16" else dims
    a_blocks, La = _batch(dims, 6, 300, dtype, 1, lengths=[300, 5, 0, 140, 260, 64])
    b_blocks, Lb = _batch(dims, 2, 200, dtype, 2, lengths=[1, 129])
    sa, sb = _session(dims, a_blocks, La, dtype), _session(dims, b_blocks, Lb, dtype)
    K = cross_gram(sa, sb, dt.DATTRI_ROUTE_FACTORED)
    N = sq_norms(sa, dt.DATTRI_ROUTE_FACTORED)
    torch.cuda.synchronize()
    ref = ocg.cross_gram(_oracle_batch(a_blocks, La), _oracle_batch(b_blocks, Lb))
    assert rel_fro(host64(K), ref) <= 1e-5
    self_ref = np.diag(ocg.cross_gram(_oracle_batch(a_blocks, La), _oracle_batch(a_blocks, La)))
    assert rel_fro(host64(N), self_ref) <= 1e-5
    assert host64(K)[2].tolist() == [0.0, 0.0] and host64(N)[2] == 0.0


@pytest.mark.parametrize("value", [float("inf"), float("nan"), 3.4e38])
def test_cross_gram_non_finite(value):
    # one value of example 1: its row of K is what float32 products give
    # (infinite or NaN, or finite where the value is), the others are untouched
    dims = [(64, 40)]
    a_blocks, _ = _batch(dims, 4, 50, "f32", 3)
    b_blocks, _ = _batch(dims, 2, 30, "f32", 4)
    a_blocks[0][1][1, 20, 7] = value * 1e-30 if np.isfinite(value) else value
    a_blocks[0][0][1, 20, 3] = 3.4e38 if np.isfinite(value) else 1.0
    sa, sb = _session(dims, a_blocks, None, "f32"), _session(dims, b_blocks, None, "f32")
    K = host64(cross_gram(sa, sb, dt.DATTRI_ROUTE_FACTORED))
    ref = ocg.cross_gram(_oracle_batch(a_blocks, None), _oracle_batch(b_blocks, None))
    keep = [0, 2, 3]
    assert rel_fro(K[keep], ref[keep]) <= 1e-5
    with np.errstate(over="ignore"):
        fits = np.isfinite(ref[1].astype(np.float32))
    assert np.array_equal(np.isfinite(K[1]), fits)
    if fits.all():
        assert rel_fro(K[1], ref[1]) <= 1e-5


@pytest.mark.parametrize("side", [0, 1])
def test_cross_gram_small_magnitudes(side):
    # one side's inputs (A or B) from ordinary size down to float32 subnormals,
    # example by example in one tile, against rows scaled up so that K stays
    # normal: every row meets the float32 bound
    scales = [1.0, 1e-30, 1e-34, 1e-36, 1e-37, 1e-40]
    dims = [(64, 40)]
    a_blocks, _ = _batch(dims, len(scales), 20, "f32", 5)
    b_blocks, _ = _batch(dims, 3, 20, "f32", 6)
    for i, s in enumerate(scales):
        a_blocks[0][side][i] *= s
    b_blocks[0][side].mul_(1e15)
    sa, sb = _session(dims, a_blocks, None, "f32"), _session(dims, b_blocks, None, "f32")
    K = host64(cross_gram(sa, sb, dt.DATTRI_ROUTE_FACTORED))
    ref = ocg.cross_gram(_oracle_batch(a_blocks, None), _oracle_batch(b_blocks, None))
    err = np.linalg.norm(K - ref, axis=1) / np.linalg.norm(ref, axis=1)
    assert np.all(err <= 1e-5), dict(zip(scales, err))


@pytest.mark.parametrize("n_layers,n,T", [(1, 2, 1040), (3, 17, 33), (70, 2, 20)])
def test_cross_gram_block_sums(n_layers, n, T):
    # block sums dealt to the reducing waves in runs of 256: one entry of many
    # runs (65 x 65 blocks, the last run short), entries of one run, more
    # entries than a wave looks up at a time, and single examples' entries
    dims = [(16, 8)] * n_layers
    a_blocks, La = _batch(dims, n, T, "f32", 7, lengths=[T - i % 3 for i in range(n)])
    b_blocks, _ = _batch(dims, 2, T, "f32", 8)
    sa, sb = _session(dims, a_blocks, La, "f32"), _session(dims, b_blocks, None, "f32")
    K, N = cross_gram(sa, sb, dt.DATTRI_ROUTE_FACTORED), sq_norms(sa, dt.DATTRI_ROUTE_FACTORED)
    ref = ocg.cross_gram(_oracle_batch(a_blocks, La), _oracle_batch(b_blocks, None))
    assert rel_fro(host64(K), ref) <= 1e-5
    assert rel_fro(host64(N), ocg.sq_norms(_oracle_batch(a_blocks, La))) <= 1e-5
