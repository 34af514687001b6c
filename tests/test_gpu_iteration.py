"""GPU parity of the Jacobi iteration at the sizes that are solved directly when the caller does not choose otherwise (33 to 640
vectors on the shorter side): it still takes over the matrices that the direct encode leaves, and those of calls that say
how it is to run.  `full_period=12` says the default and thereby keeps a call off the direct encode."""
import numpy as np
import pytest
import torch

import oracle
from paper_1806_04090_amd import binding, inputs
from gpu_common import ctx, check_svd_message_against_matrix
from test_gpu_svd import encode, full_parity
from test_gpu_svd_random import FLOOR, KINDS, make

pytestmark = pytest.mark.gpu

ITERATE = dict(full_period=12)


def iterated(n):
    return [k != (1, 2) for k in zip(ctx().svd_sweeps(n), ctx().svd_refreshes(n))]


@pytest.mark.parametrize("shape", [(33, 70), (70, 33), (64, 576), (65, 64), (96, 200), (128, 64), (160, 300), (225, 230), (256, 300),
                                   # more than four block pairs per tick; more column chunks than partial Gram matrices
                                   (300, 420), (480, 500), (72, 3300), (3200, 290),
                                   # Gram space; an odd number of blocks, an odd number of pairs
                                   (481, 481), (500, 700), (512, 600), (600, 512), (544, 600), (640, 660)])
def test_shapes(shape):
    rng = np.random.default_rng(shape[0] * 7919 + shape[1])
    G = inputs.low_rank_plus_noise(rng, shape[0], shape[1], [1.0, 0.5, 0.2], 0.02)
    msgs, per, status, _ = encode([G], 2.0, 11, stream_base=5, capacity=min(shape), **ITERATE)
    assert status == 0 and iterated(1) == [True]
    full_parity(G, 2.0, 11, 5, msgs[0], *per[0])


def test_all_kinds_in_one_call():
    shapes = [(64, 27), (64, 576), (128, 64), (10, 512), (128, 576), (256, 128), (300, 420), (512, 600), (660, 700)]
    mats = inputs.resnet18_layer_set(3, shapes=shapes)
    msgs, per, status, _ = encode(mats, 3.0, 7, stream_base=100, **ITERATE)
    assert status == 0 and [k for k, s in zip(iterated(len(shapes)), shapes) if min(s) > 32] == [True] * 7
    for j, G in enumerate(mats):
        full_parity(G, 3.0, 7, 100 + j, msgs[j], *per[j])


@pytest.mark.parametrize("kind", KINDS)
@pytest.mark.parametrize("shape", [(90, 400), (333, 250), (530, 610)])
def test_spectra(kind, shape):
    rng = np.random.default_rng(shape[0])
    G = np.ascontiguousarray(make(rng, kind, *shape), dtype=np.float32)
    msgs, per, status, _ = encode([G], 5.5, 3, stream_base=7, capacity=min(shape), max_sweeps=32, **ITERATE)
    assert status == 0
    ref = np.linalg.svd(G.astype(np.float64), compute_uv=False)
    sig, p = per[0]
    at_floor = (sig <= FLOOR * ref[0]) & (ref <= FLOOR * ref[0])
    assert (at_floor | (np.abs(sig - ref) <= 1e-4 * np.maximum(ref, 1e-3 * ref[0]))).all()
    h = msgs[0].to_host()
    assert np.array_equal(h["idx"], np.flatnonzero(oracle.bernoulli_mask(p, 3, 7)))
    check_svd_message_against_matrix(G.astype(np.float64), h, sig, p)


def test_adaptive_sweep_budget():
    shapes = [(64, 576), (256, 1152), (512, 600)]
    easy = inputs.resnet18_layer_set(21, shapes=shapes)
    want, _, status, _ = encode(easy, 3.0, 9, **ITERATE)
    assert status == 0
    want, used = [m.to_host() for m in want], ctx().svd_sweeps(len(shapes))
    assert min(used) > 1
    for _ in range(3):
        got, _, status, _ = encode(easy, 3.0, 9, adaptive=1, **ITERATE)
        assert status == 0 and ctx().svd_sweeps(len(shapes)) == used
        for a, m in zip(want, got):
            b = m.to_host()
            assert all(np.array_equal(a[k], b[k]) for k in ("idx", "w", "U", "V"))
    rng = np.random.default_rng(3)
    low = (rng.standard_normal((512, 300)) @ rng.standard_normal((300, 600))).astype(np.float32)
    assert encode([easy[0], easy[1], low], 3.0, 9, adaptive=1, **ITERATE)[2] == binding.ATOMO_ENOCONV
    assert encode([easy[0], easy[1], low], 3.0, 9, adaptive=1, **ITERATE)[2] == 0
    # a call that leaves the choice to the library learns nothing wrong from those that iterated
    for _ in range(2):
        assert encode(easy, 3.0, 9, adaptive=1)[2] == 0 and iterated(len(shapes)) == [False] * 3
    assert encode([easy[0], easy[1], low], 3.0, 9, adaptive=1, **ITERATE)[2] == 0
