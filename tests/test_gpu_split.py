"""GPU parity of the split form (stage-1 streams and the token contraction)
against the float64 oracle at the sizes where its paths change: row blocks of
256 (bf16) and 128 (float32) token rows over several examples, widths ending
inside a column stage, every map tile count of the stream, several slabs and
token chunks, lengths that leave whole row blocks unread, and float32 inputs
the three-term bf16 split cannot carry.

Products and sums are float32 on inputs held exactly, so both input types meet
the float32 bound: relative Frobenius error 1e-5 per layer block (64 float32
roundings of 6e-8 in a random walk over 4096 columns and 600 tokens stay below
5e-6)."""
import numpy as np
import pytest
import torch

import paper_2609_38767_amd as dt
import workloads as W
from gpu_util import host64, oracle_maps, oracle_phi_rows, per_layer_errors
from paper_2609_38767_amd.session import ProjectionSession

pytestmark = pytest.mark.gpu
DEV = "cuda"
TOL = 1e-5


def _layers(shapes, shared=False):
    return [dict(name=f"l{i}", d_in=a, d_out=b, k_in=ki, k_out=ko, a_group="x" if shared else f"x{i}")
            for i, (a, b, ki, ko) in enumerate(shapes)]


def _run(layers, n, T, dtype, lengths=None, seed=5, edit=None):
    wl = dict(W.WORKLOADS["tiny"], layers=layers, seed=seed)
    cache, inputs = {}, []
    for li in range(len(layers)):
        inputs.append(W.factor_blocks(wl, li, 0, n, T, DEV, dtype, a_cache=cache))
    if edit:
        edit(inputs)
    s = ProjectionSession(layers, dtype=dtype, seed=seed, form=dt.DATTRI_FORM_SPLIT)
    lens = None if lengths is None else torch.tensor(lengths, dtype=torch.int32, device=DEV)
    for li, (A, B) in enumerate(inputs):
        s.capture(li, A, B, lens)
    phi = s.project(n, route=dt.DATTRI_ROUTE_FACTORED)
    torch.cuda.synchronize()
    return inputs, host64(phi)


def _check(layers, inputs, got, n, dtype, lengths=None, seed=5):
    host = [(host64(A), host64(B)) for A, B in inputs]
    ref = oracle_phi_rows(layers, oracle_maps(seed, layers, dtype), host, list(range(n)),
                          None if lengths is None else np.asarray(lengths))
    assert np.all(np.isfinite(got))
    errs = per_layer_errors(got, ref, layers)
    assert max(errs) <= TOL, errs


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("shapes,n,T,lengths,shared", [
    # one tile; widths of one chunk and of a stage plus a chunk; a single row
    ([(8, 72, 8, 16), (40, 136, 16, 3)], 1, 1, None, False),
    # 2, 3 and 4 tiles, widths ending inside a stage; 257 rows: a second row block of one row
    ([(200, 264, 32, 48), (328, 96, 33, 64)], 1, 257, None, False),
    # 6 tiles over a shared input (q/k/v) and an 8-tile side; rows not a multiple of any block
    ([(256, 128, 32, 32), (256, 64, 32, 32), (256, 64, 32, 32)], 3, 129, None, True),
    ([(192, 320, 128, 64)], 2, 131, None, False),
    # shared inputs of 4 tiles each, merged for the stream
    ([(520, 96, 64, 64), (520, 72, 64, 64), (520, 64, 64, 64)], 2, 96, None, True),
    # whole row blocks past every length, empty and full examples, one row
    ([(136, 520, 64, 32)], 5, 300, [0, 300, 1, 17, 256], False),
    # few workgroups over long sequences: token chunks and their reduction; several slabs
    ([(4104, 64, 16, 16)], 2, 1100, [1100, 513], False),
    # the first length that is cut into chunks: the last one of a single token, an example ending in each chunk
    ([(64, 96, 32, 64)], 3, 257, [257, 128, 129], False),
    ([(72, 64, 128, 64)], 2, 520, None, False),
    # fewer rows than map columns: slabs set by the map's width
    ([(4104, 1032, 64, 64), (4104, 2056, 16, 16)], 1, 20, [17], False),
])
def test_split_stream_edges(dtype, shapes, n, T, lengths, shared):
    layers = _layers(shapes, shared)
    inputs, got = _run(layers, n, T, dtype, lengths)
    _check(layers, inputs, got, n, dtype, lengths)


def test_split_stream_wide_values():
    # magnitudes over 30 decades in one row: every split term stays normal, and
    # the largest entries of phi (about 1e15 x 1e15 x 40 tokens) stay finite in float32
    layers = _layers([(96, 160, 32, 32)])

    def edit(inputs):
        for X in inputs[0]:
            e = torch.linspace(-15, 15, X.shape[-1], device=DEV)
            X.mul_(torch.pow(10.0, e)[torch.randperm(X.shape[-1], device=DEV)])

    inputs, got = _run(layers, 2, 40, "f32", edit=edit)
    _check(layers, inputs, got, 2, "f32")


@pytest.mark.parametrize("value", [float("inf"), float("-inf"), float("nan"), 3.4e38])
def test_split_stream_non_finite(value):
    # a value the bf16 split cannot carry leaves its own row's projections as
    # float32 products give them: the phi of its example is what float32 torch
    # gives (infinite, NaN or huge in the same places), others are untouched
    layers = _layers([(64, 96, 16, 16)])

    def edit(inputs):
        inputs[0][0][1, 7, 5] = value

    inputs, got = _run(layers, 3, 24, "f32", edit=edit)
    A, B = (x.double().cpu() for x in inputs[0])
    P_in, P_out = (torch.from_numpy(np.asarray(m, dtype=np.float64)) for m in oracle_maps(5, layers, "f32")[0])
    rows = (A[1] @ P_in).float().double()  # the projected rows are float32
    ref = (rows.t() @ (B[1] @ P_out)).reshape(-1).numpy()
    with np.errstate(over="ignore"):
        ref = ref.astype(np.float32).astype(np.float64)
    same = np.isfinite(ref)
    assert np.array_equal(np.isfinite(got[1]), same)
    if same.any():
        assert np.linalg.norm(got[1][same] - ref[same]) <= TOL * np.linalg.norm(ref[same])
    host = [(host64(X), host64(Y)) for X, Y in inputs]
    clean = oracle_phi_rows(layers, oracle_maps(5, layers, "f32"), host, [0, 2], None)
    assert max(per_layer_errors(got[[0, 2]], clean, layers)) <= TOL


def test_split_stream_small_magnitudes():
    # examples of one token, from ordinary size down to float32 subnormals, side
    # by side in one row block (the other side scaled so that phi stays normal):
    # each block meets the float32 bound.  Sums of subnormal results round at
    # 2^-150: 96 of them in a result of about 1e-40 stay below 1e-3 of it.
    scales = [1.0, 1e-30, 1e-34, 1e-36, 1e-37, 1e-40, 0.0, 1.0]
    layers = _layers([(96, 160, 32, 48)])

    def edit(inputs):
        for i, s in enumerate(scales):
            inputs[0][0][i] *= s
            inputs[0][1][i] *= 1e15 if 0.0 < s < 1e-20 else 1.0

    inputs, got = _run(layers, len(scales), 1, "f32", edit=edit)
    host = [(host64(A), host64(B)) for A, B in inputs]
    ref = oracle_phi_rows(layers, oracle_maps(5, layers, "f32"), host, list(range(len(scales))), None)
    errs = {s: np.linalg.norm(got[i] - ref[i]) / max(np.linalg.norm(ref[i]), 1e-300) for i, s in enumerate(scales)}
    assert all(e <= (TOL if s == 0.0 or s > 1e-38 else 1e-3) for s, e in errs.items()), errs


@pytest.mark.parametrize("side", [0, 1])
def test_split_stream_small_maps(side):
    # a map column too small to split beside ordinary ones
    shape, seed, n, T = dict(d_in=64, d_out=96, k_in=16, k_out=16), 7, 3, 20
    maps = [np.random.default_rng(seed).standard_normal((d, 16)).astype(np.float32) for d in (64, 96)]
    maps[side][:, 5] *= 1e-36
    s = ProjectionSession([shape], dtype="f32", seed=seed, form=dt.DATTRI_FORM_SPLIT, overrides={0: tuple(maps)})
    g = torch.Generator(device=DEV).manual_seed(seed)
    A, B = (torch.randn((n, T, d), generator=g, device=DEV) * 1e2 for d in (64, 96))
    s.capture(0, A, B)
    got = host64(s.project(n, route=dt.DATTRI_ROUTE_FACTORED)).reshape(n, 16, 16)
    a, b = (X.double().cpu().numpy() @ m.astype(np.float64) for X, m in zip((A, B), maps))
    ref = np.einsum("itc,itr->icr", a, b)
    for c in (5, 6):  # the small column and an ordinary one
        x, y = (got[:, c], ref[:, c]) if side == 0 else (got[:, :, c], ref[:, :, c])
        assert np.linalg.norm(x - y) <= TOL * np.linalg.norm(y)
