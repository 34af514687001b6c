"""GPU parity: atomo_decode fed oracle-made messages."""
import numpy as np
import pytest
import torch

import oracle
from paper_1806_04090_amd import binding
from gpu_common import ctx, dev

pytestmark = pytest.mark.gpu


def make_msg(rng, rows, cols, k, capacity):
    host = {"w": rng.standard_normal(k), "U": rng.standard_normal((rows, k)), "V": rng.standard_normal((cols, k))}
    m = binding.alloc_svd_message(rows, cols, capacity, "cuda")
    m.count.fill_(k)
    m.idx[:k] = torch.arange(k, dtype=torch.int32)
    m.w[:k] = dev(host["w"].astype(np.float32))
    m.U[:k] = dev(host["U"].T.astype(np.float32))
    m.V[:k] = dev(host["V"].T.astype(np.float32))
    host = {key: val.astype(np.float32).astype(np.float64) for key, val in host.items()}
    return m, host


@pytest.mark.parametrize("rows,cols,ks", [(1, 1, [1]), (5, 7, [3]), (64, 576, [2]), (70, 300, [0, 4, 1]),
                                          (130, 1030, [3, 3, 2, 5]), (512, 4608, [3]), (10, 512, [48])])
def test_svd_decode_matches_oracle(rows, cols, ks):
    rng = np.random.default_rng(rows * 31 + cols)
    pairs = [make_msg(rng, rows, cols, k, max(k, 1) + 2) for k in ks]
    scale = 1.0 / len(ks)
    out = binding.atomo_decode(ctx(), [m for m, _ in pairs], scale=scale).cpu().numpy()
    want = oracle.decode_svd([h for _, h in pairs], rows, cols, scale=scale)
    assert np.linalg.norm(out - want) <= 1e-5 * max(np.linalg.norm(want), 1e-30)
    np.testing.assert_allclose(out, want, rtol=0, atol=1e-5 * max(np.abs(want).max(), 1e-30))


@pytest.mark.parametrize("rows,cols,capacity,ks", [(40, 130, 100, [7, 0, 99, 100, 1, 33, 2, 2, 2, 50, 5, 64]),   # batches of 5 messages
                                                   (96, 70, 512, [512, 3]),                                     # the atom list is staged in two pieces
                                                   (600, 600, 600, [600]),                                      # every atom of a 600 x 600 matrix kept (p = 1)
                                                   (130, 2048, 130, [130, 129, 1]),
                                                   (33, 33, 6, [5] * 90)])                                      # 85 messages per batch, then 5
def test_svd_decode_many_messages_across_batches(rows, cols, capacity, ks):
    rng = np.random.default_rng(len(ks) * 7 + rows)
    pairs = [make_msg(rng, rows, cols, k, capacity) for k in ks]
    out = binding.atomo_decode(ctx(), [m for m, _ in pairs], scale=0.5).cpu().numpy()
    want = oracle.decode_svd([h for _, h in pairs], rows, cols, scale=0.5)
    assert np.linalg.norm(out - want) <= 1e-5 * max(np.linalg.norm(want), 1e-30)


@pytest.mark.parametrize("messages,capacity", [(2, 256), (16, 32), (17, 30), (63, 8), (64, 8), (65, 7), (129, 3), (512, 1)])
def test_svd_decode_lists_of_messages(messages, capacity):
    """A wave lists 64 messages at a time, one scan over their counts; some keep nothing, some all they can.  An entry of the result is a
    sum of K products in float: its error is at most (K + 2) eps times the sum of their magnitudes."""
    rng = np.random.default_rng(messages)
    ks = [int(k) for k in rng.integers(0, capacity + 1, messages)]
    ks[0], ks[-1] = 0, capacity
    pairs = [make_msg(rng, 5, 36, k, capacity) for k in ks]
    out = binding.atomo_decode(ctx(), [m for m, _ in pairs]).cpu().numpy()
    want = oracle.decode_svd([h for _, h in pairs], 5, 36)
    size = oracle.decode_svd([{key: np.abs(x) for key, x in h.items()} for _, h in pairs], 5, 36)
    assert (np.abs(out - want) <= (sum(ks) + 2) * 2.0 ** -24 * size).all()


@pytest.mark.parametrize("rows,cols", [(64, 256), (33, 300), (300, 18)])
@pytest.mark.parametrize("k", [1, 2, 3, 16, 17, 33])
@pytest.mark.parametrize("scale", [np.inf, -np.inf])
def test_svd_decode_with_an_infinite_scale(rows, cols, k, scale):
    """Atoms of positive entries: every element of the sum is infinite, for odd and even numbers of atoms alike."""
    rng = np.random.default_rng(k)
    m, _ = make_msg(rng, rows, cols, k, k + 1)
    for part in (m.w, m.U, m.V):
        part[:k] = part[:k].abs() + 0.5
    out = binding.atomo_decode(ctx(), [m], scale=scale)
    assert (out == scale).all()
    binding.atomo_apply_svd_batch(ctx(), [[m]], scale, [out])
    assert (out == scale).all()


def test_svd_decode_into_strided_output_and_batch():
    rng = np.random.default_rng(1)
    m1, h1 = make_msg(rng, 33, 50, 2, 4)
    m2, h2 = make_msg(rng, 70, 20, 3, 4)
    big = torch.full((33, 64), 7.0, device="cuda")
    binding.atomo_decode(ctx(), [m1], out=big[:, 3:53])
    got = big.cpu().numpy()
    np.testing.assert_allclose(got[:, 3:53], oracle.decode_svd([h1], 33, 50), rtol=1e-5, atol=1e-5)
    assert (got[:, :3] == 7).all() and (got[:, 53:] == 7).all()
    outs = binding.atomo_decode_svd_batch(ctx(), [[m1], [m2]])
    np.testing.assert_allclose(outs[0].cpu().numpy(), oracle.decode_svd([h1], 33, 50), rtol=1e-5, atol=1e-5)
    np.testing.assert_allclose(outs[1].cpu().numpy(), oracle.decode_svd([h2], 70, 20), rtol=1e-5, atol=1e-5)


def test_entrywise_decode_matches_oracle():
    rng = np.random.default_rng(2)
    n = 10_007
    msgs, hosts = [], []
    for k in (0, 1, 500):
        idx = np.sort(rng.choice(n, size=k, replace=False))
        val = rng.standard_normal(k).astype(np.float32)
        m = binding.alloc_entrywise_message(n, max(k, 1), "cuda")
        m.count.fill_(k)
        if k:
            m.idx[:k] = dev(idx.astype(np.uint32).view(np.int32))
            m.val[:k] = dev(val)
        msgs.append(m); hosts.append({"idx": idx, "val": val.astype(np.float64)})
    out = binding.atomo_decode(ctx(), msgs, scale=0.5).cpu().numpy()
    np.testing.assert_allclose(out, oracle.decode_entrywise(hosts, n, scale=0.5), rtol=1e-6, atol=1e-9)


def test_matrix_core_rate_probe_returns_a_plausible_figure():
    # the measurement helper of bench.py: between a tenth of and the whole published fp32 matrix-core peak
    rate = ctx().measure_mfma_fp32()
    assert 15.0 < rate < 160.0


@pytest.mark.parametrize("accumulate", [False, True])
def test_svd_decode_of_tall_and_other_outputs_in_one_call(accumulate):
    """Outputs of at most 32 columns have tiles of their own in the same launch: both kinds, their edges, unaligned rows, several
    messages and none that keeps anything.  An entry is a sum of K products in float, and one more with what was there: its error is at
    most (K + 4) eps times the sum of the magnitudes."""
    rng = np.random.default_rng(5)
    shapes = [(64, 576), (1, 1), (2049, 18), (300, 32), (300, 33), (4097, 2), (33, 31), (130, 1030), (5000, 17), (513, 27)]
    scale = 0.375
    groups, outs, starts = [], [], []
    for j, (rows, cols) in enumerate(shapes):
        groups.append([make_msg(rng, rows, cols, k, 6) for k in ([3], [0, 4, 1], [0])[j % 3]])
        ld = cols + j % 4
        start = rng.standard_normal((rows, ld)).astype(np.float32)
        starts.append(start)
        outs.append(dev(start)[:, :cols])
    messages = [[m for m, _ in grp] for grp in groups]
    if accumulate:
        binding.atomo_apply_svd_batch(ctx(), messages, scale, outs)
    else:
        binding.atomo_decode_svd_batch(ctx(), messages, scale, outs=outs)
    for (rows, cols), grp, out, start in zip(shapes, groups, outs, starts):
        want = oracle.decode_svd([h for _, h in grp], rows, cols, scale=scale)
        size = oracle.decode_svd([{key: np.abs(x) for key, x in h.items()} for _, h in grp], rows, cols, scale=scale)
        if accumulate:
            want = want + start[:, :cols]
            size = size + np.abs(start[:, :cols])
        terms = sum(h["w"].size for _, h in grp)
        assert (np.abs(out.cpu().numpy() - want) <= (terms + 4) * 2.0 ** -23 * size).all(), (rows, cols)


@pytest.mark.parametrize("offset", [0, 1, 2])                    # (aligned to 16, 4 and 8 bytes)
@pytest.mark.parametrize("rows,cols", [(65, 1), (256, 2), (257, 17), (511, 18), (700, 24), (700, 25), (300, 32)])
def test_svd_decode_of_narrow_outputs_without_gaps(rows, cols, offset):
    """Tiles of up to 24 columns leave through LDS as one piece of memory; what lies before and behind the output stays.  Tolerance as above."""
    rng = np.random.default_rng(rows + cols)
    for ks in ([3], [0], [2, 0, 17]):
        pairs = [make_msg(rng, rows, cols, k, 20) for k in ks]
        flat = torch.full((rows * cols + 16,), 7.5, device="cuda")
        out = flat[offset:offset + rows * cols].view(rows, cols)
        binding.atomo_decode_svd_batch(ctx(), [[m for m, _ in pairs]], 0.5, outs=[out])
        want = oracle.decode_svd([h for _, h in pairs], rows, cols, scale=0.5)
        size = oracle.decode_svd([{key: np.abs(x) for key, x in h.items()} for _, h in pairs], rows, cols, scale=0.5)
        assert (np.abs(out.cpu().numpy() - want) <= (sum(ks) + 4) * 2.0 ** -23 * size).all()
        assert bool((flat[:offset] == 7.5).all()) and bool((flat[offset + rows * cols:] == 7.5).all())


@pytest.mark.parametrize("rows,cols,gap", [(256, 25, 0), (512, 32, 0), (769, 31, 0), (255, 28, 0), (512, 18, 3), (600, 24, 1), (256, 1, 1), (1025, 32, 5)])
def test_svd_decode_of_tall_tiles_that_are_not_one_piece_of_memory(rows, cols, gap):
    """More than 24 columns, or gaps between the rows: whole tiles and the last one.  What lies between and behind the rows stays.  Tolerance as above."""
    rng = np.random.default_rng(rows + cols)
    for ks in ([3], [0], [2, 0, 17]):
        pairs = [make_msg(rng, rows, cols, k, 20) for k in ks]
        flat = torch.full((rows + 2, cols + gap), 7.5, device="cuda")
        out = flat[1:rows + 1, :cols]
        binding.atomo_decode_svd_batch(ctx(), [[m for m, _ in pairs]], 0.5, outs=[out])
        want = oracle.decode_svd([h for _, h in pairs], rows, cols, scale=0.5)
        size = oracle.decode_svd([{key: np.abs(x) for key, x in h.items()} for _, h in pairs], rows, cols, scale=0.5)
        assert (np.abs(out.cpu().numpy() - want) <= (sum(ks) + 4) * 2.0 ** -23 * size).all()
        assert bool((flat[0] == 7.5).all()) and bool((flat[rows + 1] == 7.5).all()) and bool((flat[:, cols:] == 7.5).all())


def test_more_than_24_columns_take_no_longer_for_the_form_of_fewer():
    # 600,000 rows: 25 columns took 1.14 times as long as 24 with the form for up to 24 in the same kernel, 0.97 times without it
    rng, times = np.random.default_rng(3), []
    for cols in (24, 25):
        pairs = [make_msg(rng, 600_000, cols, 3, 3) for _ in range(4)]
        out = torch.zeros(600_000, cols, device="cuda")
        took = []
        for _ in range(15):
            start, end = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            start.record()
            for _ in range(20):
                binding.atomo_decode_svd_batch(ctx(), [[m for m, _ in pairs]], 1.0, outs=[out])
            end.record()
            end.synchronize()
            took.append(start.elapsed_time(end))
        times.append(min(took))
    assert times[1] < 1.09 * times[0], times
