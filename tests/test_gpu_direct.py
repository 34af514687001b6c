"""GPU parity of the direct encode (Gram matrix, tridiagonal form, eigenvectors of the kept atoms): the edges of its size
classes and tiles against the fp64 oracle, and the cases that it leaves to the Jacobi iteration."""
import numpy as np
import pytest
import torch

import oracle
from paper_1806_04090_amd import binding, inputs
from gpu_common import ctx, dev, check_svd_message_against_matrix
from test_gpu_svd import encode, full_parity

pytestmark = pytest.mark.gpu

DIRECT = (1, 2)                                                  # sweeps and passes over the data that it reports


def route(n=1):
    return list(zip(ctx().svd_sweeps(n), ctx().svd_refreshes(n)))


@pytest.mark.parametrize("shape", [(33, 33), (40, 63), (64, 1300), (65, 70), (127, 128), (128, 129), (129, 131), (192, 257),
                                   (255, 256), (256, 300), (257, 258), (448, 449), (511, 512), (512, 513), (513, 520),
                                   (576, 577), (577, 600), (639, 641), (640, 640)])
@pytest.mark.parametrize("tall", [False, True])
def test_sizes_around_the_tiles(shape, tall):
    rng = np.random.default_rng(shape[0] * 1009 + shape[1])
    m, n = shape[::-1] if tall else shape
    # (a square of noise has one singular value near zero: let it stay above the floor)
    G = inputs.low_rank_plus_noise(rng, m, n, [1.0, 0.5, 0.25, 0.1], 0.01)
    msgs, per, status, sweeps = encode([G], 3.0, 5, stream_base=3, capacity=min(shape))
    assert status == 0
    if abs(m - n) > 8:
        assert route() == [DIRECT]
    full_parity(G, 3.0, 5, 3, msgs[0], *per[0])


@pytest.mark.parametrize("shape", [(34, 90), (47, 80), (48, 300), (49, 100), (79, 120), (80, 96), (81, 200), (95, 130), (96, 400),
                                   (97, 150), (111, 160), (112, 300), (113, 140), (126, 180), (130, 300), (160, 200), (193, 240),
                                   (321, 400), (384, 420), (385, 500)])
def test_sizes_around_the_slots_of_one_workgroup(shape):
    """Slots of 16 rows, steps on the same slots in runs of 32; behind a group the last rows of an even or odd number of chunks."""
    rng = np.random.default_rng(shape[0] * 2003 + shape[1])
    G = inputs.low_rank_plus_noise(rng, *shape, [1.0, 0.5, 0.25, 0.1], 0.01)
    msgs, per, status, sweeps = encode([G], 3.0, 7, stream_base=2, capacity=min(shape))
    assert status == 0 and route() == [DIRECT]
    full_parity(G, 3.0, 7, 2, msgs[0], *per[0])


def test_strided_folded_and_mixed_with_other_sizes_in_one_call():
    rng = np.random.default_rng(3)
    shapes = [(64, 27), (96, 200), (650, 660), (300, 140), (512, 700)]
    host = [inputs.low_rank_plus_noise(rng, m, n, [1.0, 0.4, 0.2], 0.01) for m, n in shapes]
    mats = []
    for g in host:
        wide = torch.zeros(g.shape[0], g.shape[1] + 3, device="cuda")
        wide[:, 1:-2] = dev(g)
        mats.append(wide[:, 1:-2])                               # rows that start anywhere, an odd stride
    total = sum(min(s) for s in shapes)
    sigma, p = torch.zeros(total, device="cuda"), torch.zeros(total, device="cuda")
    plain = binding.atomo_encode_svd(ctx(), mats, 3.0, 9, 40, sigma_out=sigma, p_out=p)
    assert ctx().status()[0] == 0
    kinds = route(len(shapes))
    assert [k == DIRECT for k in kinds[1:]] == [True, False, True, True]
    folded = [binding.alloc_svd_message(m, n, binding.default_capacity(3.0, min(m, n)), "cuda", folded=True) for m, n in shapes]
    binding.atomo_encode_svd(ctx(), mats, 3.0, 9, 40, msgs=folded)
    assert ctx().status()[0] == 0
    a = binding.atomo_decode_svd_batch(ctx(), [[m] for m in plain])
    b = binding.atomo_decode_svd_batch(ctx(), [[m] for m in folded])
    at = 0
    for j, g in enumerate(host):
        r = min(g.shape)
        full_parity(g, 3.0, 9, 40 + j, plain[j], sigma[at:at + r].cpu().numpy(), p[at:at + r].cpu().numpy())
        at += r
        assert torch.linalg.norm(a[j] - b[j]) <= 1e-5 * torch.linalg.norm(a[j])


@pytest.mark.parametrize("shape", [(100, 300), (300, 400), (600, 620)])
def test_left_to_the_iteration(shape):
    # rank below the shorter side, kept atoms with equal singular values, an explicit option, a budget of many atoms
    rng = np.random.default_rng(shape[0])
    m, n = shape
    low = (rng.standard_normal((m, m // 2)) @ rng.standard_normal((m // 2, n))).astype(np.float32)
    q, _ = np.linalg.qr(rng.standard_normal((n, m)))
    equal = np.zeros((m, n), dtype=np.float32)
    equal[:, :m] = np.eye(m, dtype=np.float32)                   # every singular value is 1
    for G, kw, s in ((low, {}, 3.0), (equal, {}, 32.0), (q.T.astype(np.float32), dict(block_order=1), 3.0),
                     (q.T.astype(np.float32), {}, 40.0)):
        msgs, per, status, _ = encode([G], s, 2, capacity=m, **kw)
        assert status == 0 and route() != [DIRECT]
        check_svd_message_against_matrix(G.astype(np.float64), msgs[0].to_host(), *per[0])


@pytest.mark.parametrize("shape", [(120, 300), (500, 400)])
def test_rows_of_zeros_and_a_matrix_of_zeros_are_solved_directly(shape):
    # filters that got no gradient: as many singular values are exactly zero
    rng = np.random.default_rng(shape[1])
    G = inputs.low_rank_plus_noise(rng, *shape, [1.0, 0.5], 0.02)
    dead = rng.choice(min(shape), 17, replace=False)
    if shape[0] < shape[1]:
        G[dead] = 0
    else:
        G[:, dead] = 0
    msgs, per, status, _ = encode([G, np.zeros(shape, dtype=np.float32)], 3.0, 4, capacity=16)
    assert status == 0 and route(2) == [DIRECT, DIRECT]
    assert (per[0][0][-17:] == 0).all() and (per[0][1][-17:] == 0).all() and (per[0][0][:-17] > 0).all()
    full_parity(G, 3.0, 4, 0, msgs[0], *per[0])
    assert (per[1][0] == 0).all() and msgs[1].to_host()["count"] == 0


def test_many_matrices_in_one_call_give_the_bits_of_calls_of_their_own():
    # more groups than run at once, another number of points per eigenvalue
    shapes = [(512, 520)] * 40 + [(96, 130)] * 40 + [(530, 600)] * 3
    host = [inputs.low_rank_plus_noise(np.random.default_rng(j % 2), m, n, [1.0, 0.3], 0.02) for j, (m, n) in enumerate(shapes)]
    mats = [dev(g) for g in host]
    ids = [7 + j % 2 for j in range(len(shapes))]
    many = binding.atomo_encode_svd(ctx(), mats, 3.0, 1, 0, stream_ids=ids)
    assert ctx().status()[0] == 0
    for j in (0, 1, 39, 40, 79, 80, 82):
        one = binding.atomo_encode_svd(ctx(), [mats[j]], 3.0, 1, ids[j])[0].to_host()
        got = many[j].to_host()
        assert got["count"] == one["count"] and all(np.array_equal(got[k], one[k]) for k in ("idx", "w", "U", "V")), j
    assert ctx().status()[0] == 0


def test_calls_of_many_gram_tiles_give_the_bits_of_calls_of_their_own():
    """From 8192 work items of the Gram product on, whole tiles of wide matrices in chunks of 256 columns and more are a wave's; tall, padded
    and odd ones and shorter chunks beside them."""
    gen = torch.Generator(device="cuda").manual_seed(11)
    shapes = [(512, 2048)] * 30 + [(2048, 512), (500, 2048), (512, 2041), (449, 2064), (64, 640), (512, 1152)]
    mats = []
    for m, n in shapes:
        wide = torch.randn(m, n + 3, generator=gen, device="cuda") * 0.01
        wide[0] *= 40.0
        mats.append(wide[:, 1:n + 1])                            # rows that start anywhere
    total = sum(min(s) for s in shapes)
    sigma = torch.zeros(total, device="cuda")
    many = binding.atomo_encode_svd(ctx(), mats, 3.0, 4, 70, sigma_out=sigma)
    assert ctx().status()[0] == 0 and route(len(shapes)) == [DIRECT] * len(shapes)
    for j in (0, 13, 29, 30, 31, 32, 33, 34, 35):
        r, at = min(shapes[j]), sum(min(s) for s in shapes[:j])
        own = torch.zeros(r, device="cuda")
        one = binding.atomo_encode_svd(ctx(), [mats[j]], 3.0, 4, 70 + j, sigma_out=own)[0]
        assert ctx().status()[0] == 0
        assert torch.equal(own, sigma[at:at + r])
        a, b = one.to_host(), many[j].to_host()
        assert a["count"] == b["count"] and all(np.array_equal(a[k], b[k]) for k in ("idx", "w", "U", "V")), j


def test_calls_of_many_gram_tiles_one_after_the_other():
    """A training loop: the descriptors of the first call are found on the device by the others, which have other numbers in the same
    buffers, and each call counts the parts of its Gram matrices from nothing."""
    gen = torch.Generator(device="cuda").manual_seed(12)
    mats = [torch.empty(512, 2048, device="cuda") for _ in range(31)] + [torch.empty(200, 300, device="cuda")]
    msgs = None
    for step in range(4):
        for g in mats:
            g.copy_(torch.randn(g.shape, generator=gen, device="cuda") * 0.01)
            g[step] *= 40.0
        msgs = binding.atomo_encode_svd(ctx(), mats, 3.0, step, 70, msgs=msgs, adaptive=1)
        assert ctx().status()[0] == 0 and route(len(mats)) == [DIRECT] * len(mats)
        for j in (0, 17, 30, 31):
            one = binding.atomo_encode_svd(ctx(), [mats[j]], 3.0, step, 70 + j)[0]
            a, b = one.to_host(), msgs[j].to_host()
            assert a["count"] == b["count"] and all(np.array_equal(a[k], b[k]) for k in ("idx", "w", "U", "V")), (step, j)


def test_beside_the_work_of_another_stream():
    """Groups find their places among other workgroups, or give up in bounded time and are reduced alone: a message either way."""
    shapes = [(512, 700), (300, 400), (129, 260), (64, 100), (900, 18)]
    host = [inputs.low_rank_plus_noise(np.random.default_rng(j), m, n, [1.0, 0.3], 0.02) for j, (m, n) in enumerate(shapes)]
    mats = [dev(g) for g in host]
    a, c = torch.ones(4096, 4096, device="cuda"), torch.empty(4096, 4096, device="cuda")
    one, two = torch.cuda.Stream(), torch.cuda.Stream()
    want = [m.to_host() for m in binding.atomo_encode_svd(ctx(), mats, 3.0, 6, 90)]
    torch.cuda.synchronize()
    for adaptive in (0, 1, 1, 1):
        with torch.cuda.stream(two):
            for _ in range(3):
                torch.mm(a, a, out=c)
        msgs = binding.atomo_encode_svd(ctx(), mats, 3.0, 6, 90, adaptive=adaptive, stream=one)
        one.synchronize()
        assert ctx().status(one)[0] == 0
        for m, w in zip(msgs, want):
            got = m.to_host()
            assert got["count"] == w["count"] and np.array_equal(got["idx"], w["idx"])
            np.testing.assert_allclose(got["w"], w["w"], rtol=1e-6)
    torch.cuda.synchronize()


def test_a_training_loop_enqueues_the_direct_encode_alone_until_it_falls_short():
    shape = (200, 260)
    rng = np.random.default_rng(0)
    easy = inputs.low_rank_plus_noise(rng, *shape, [1.0, 0.5], 0.02)
    low = (rng.standard_normal((shape[0], 50)) @ rng.standard_normal((50, shape[1]))).astype(np.float32)
    want = encode([easy], 3.0, 9)[0][0].to_host()
    for _ in range(3):
        msgs, per, status, _ = encode([easy], 3.0, 9, adaptive=1)
        got = msgs[0].to_host()
        assert status == 0 and all(np.array_equal(got[k], want[k]) for k in ("idx", "w", "U", "V"))
    msgs, per, status, _ = encode([low], 3.0, 9, adaptive=1)
    assert status == binding.ATOMO_ENOCONV
    check_svd_message_against_matrix(low.astype(np.float64), msgs[0].to_host(), *per[0])
    msgs, per, status, _ = encode([low], 3.0, 9, adaptive=1)
    assert status == 0 and route() != [DIRECT]


def nearly_equal_tail(rng, m, n, tail):
    """One dominant singular value over a tail of equal ones, which the rounding to fp32 pulls apart by about 1e-8."""
    u, _ = np.linalg.qr(rng.standard_normal((m, min(m, n))))
    v, _ = np.linalg.qr(rng.standard_normal((n, min(m, n))))
    s = np.full(min(m, n), tail)
    s[0] = 1.0
    return ((u * s) @ v.T).astype(np.float32)


@pytest.mark.parametrize("tail", [1e-2, 1e-3, 1e-4, 1e-5])
@pytest.mark.parametrize("shape", [(60, 80), (120, 100), (300, 400), (560, 520)])
def test_kept_vectors_of_a_nearly_equal_tail_are_orthogonal(shape, tail):
    # neighbours that the search tells apart but a vector with a residual that is small against the largest eigenvalue
    # does not: accepted, they had cosines of 0.1 and more
    r = min(shape)
    host = [nearly_equal_tail(np.random.default_rng(seed), *shape, tail) for seed in range(4)]
    msgs, per, status, _ = encode(host, 32.0, 1, capacity=r)
    assert status == 0
    for G, msg, (sigma, p) in zip(host, msgs, per):
        check_svd_message_against_matrix(G.astype(np.float64), msg.to_host(), sigma, p)


@pytest.mark.parametrize("shapes", [[(660, 700)], [(200, 260), (660, 700), (300, 18)]])
def test_the_sweep_budget_of_matrices_that_iterate_beside_solved_ones_is_kept(shapes):
    # a budget in force shows in a gradient that needs more sweeps than it allows; from the third call on the
    # launches of all sweeps were enqueued again
    rng = np.random.default_rng(1)
    easy = [inputs.low_rank_plus_noise(rng, m, n, [1.0, 0.5], 0.02) for m, n in shapes]
    big = shapes.index((660, 700))
    low = (rng.standard_normal((660, 300)) @ rng.standard_normal((300, 700))).astype(np.float32)
    hard = [low if j == big else g for j, g in enumerate(easy)]
    assert encode(easy, 3.0, 9)[2] == 0
    used = ctx().svd_sweeps(len(shapes))[big]
    assert encode(hard, 3.0, 9)[2] == 0 and ctx().svd_sweeps(len(shapes))[big] > used + 1
    for _ in range(4):
        assert encode(easy, 3.0, 9, adaptive=1)[2] == 0
    assert encode(hard, 3.0, 9, adaptive=1)[2] == binding.ATOMO_ENOCONV
    assert encode(hard, 3.0, 9, adaptive=1)[2] == 0


def test_sweep_counts_of_calls_that_solved_a_matrix_directly_are_no_budget_for_its_iteration():
    shapes = [(200, 260), (660, 700)]
    rng = np.random.default_rng(2)
    easy = [inputs.low_rank_plus_noise(rng, m, n, [1.0, 0.5], 0.02) for m, n in shapes]
    quick = np.zeros(shapes[1], dtype=np.float32)
    quick[:, :660] = np.diag(np.linspace(1, 2, 660))             # orthogonal rows: done in the first sweep
    low = (rng.standard_normal((200, 120)) @ rng.standard_normal((120, 260))).astype(np.float32)
    for _ in range(3):
        assert encode([easy[0], quick], 3.0, 9, adaptive=1)[2] == 0
    assert encode([low, quick], 3.0, 9, adaptive=1)[2] == binding.ATOMO_ENOCONV
    assert encode([low, quick], 3.0, 9, adaptive=1)[2] == 0      # (now it iterates, with all sweeps)
    for _ in range(2):
        assert encode([easy[0], quick], 3.0, 9, adaptive=1)[2] == 0
    assert encode([easy[0], quick], 40.0, 9, adaptive=1)[2] == 0     # a budget of many atoms: everything iterates


def test_a_matrix_that_was_turned_down_iterates_without_another_attempt_and_is_tried_again_later():
    shapes = [(200, 260), (300, 320), (96, 18), (70, 90)]
    rng = np.random.default_rng(5)
    easy = [inputs.low_rank_plus_noise(rng, m, n, [1.0, 0.5], 0.02) for m, n in shapes]
    low = (rng.standard_normal((300, 90)) @ rng.standard_normal((90, 320))).astype(np.float32)
    poor = [easy[0], low, easy[2], easy[3]]
    want = [m.to_host() for m in encode(poor, 3.0, 9)[0]]
    solved = lambda: [k == DIRECT for k in route(len(shapes))]
    for _ in range(3):
        msgs, _, status, _ = encode(poor, 3.0, 9, adaptive=1)
        assert status == 0 and solved() == [True, False, True, True]
        for a, m in zip(want, msgs):
            b = m.to_host()
            assert all(np.array_equal(a[k], b[k]) for k in ("idx", "w", "U", "V"))
    # a gradient of full rank in its place: iterates for a while (the others have no iteration behind them), then is solved
    took = 0
    while True:
        msgs, per, status, _ = encode(easy, 3.0, 9, adaptive=1)
        assert status == 0
        full_parity(easy[1], 3.0, 9, 1, msgs[1], *per[1])
        if all(solved()):
            break
        took += 1
    assert 3 <= took <= 8
    # a budget of many atoms in between: no attempt, no history from it, and none lost
    assert encode(easy, 40.0, 9, adaptive=1)[2] == 0
    assert encode(easy, 3.0, 9, adaptive=1)[2] == 0 and all(solved())


@pytest.mark.parametrize("shapes", [[(660, 700), (200, 260), (512, 600)],                        # no data-space matrix iterates
                                    [(660, 700), (300, 400), (200, 260), (300, 18)],             # large ones do
                                    [(660, 700), (300, 400), (96, 130), (200, 260), (300, 18)],  # and small ones: no free stream
                                    [(300, 400), (96, 130), (200, 260)]])
def test_matrices_solved_beside_the_iteration_of_others_give_the_same_bits(shapes):
    rng = np.random.default_rng(6)
    host = [inputs.low_rank_plus_noise(rng, m, n, [1.0, 0.5], 0.02) for m, n in shapes]
    for j, (m, n) in enumerate(shapes):
        if (m, n) in ((300, 400), (96, 130)):                    # low rank: they iterate
            host[j] = (rng.standard_normal((m, 40)) @ rng.standard_normal((40, n))).astype(np.float32)
    want, per_want, status, _ = encode(host, 3.0, 9)
    assert status == 0
    want = [m.to_host() for m in want]
    for _ in range(5):
        msgs, per, status, _ = encode(host, 3.0, 9, adaptive=1)
        assert status == 0
        for a, m, x, y in zip(want, msgs, per_want, per):
            b = m.to_host()
            assert all(np.array_equal(a[k], b[k]) for k in ("idx", "w", "U", "V")) and np.array_equal(x, y)


@pytest.fixture
def groups():
    yield ctx().debug_direct_groups
    ctx().debug_direct_groups()


@pytest.mark.parametrize("shape", [(129, 140), (200, 300), (256, 300), (300, 257), (512, 600), (530, 513), (640, 660)])
def test_groups_over_several_dies_and_groups_that_do_not_come_together(groups, shape):
    host = [inputs.low_rank_plus_noise(np.random.default_rng(seed), *shape, [1.0, 0.5, 0.2], 0.02) for seed in range(3)]
    host[2][:, 5:9] = 0                                          # (a few rows or columns of zeros)
    host[2][5:9] = 0
    want, per_want, status, _ = encode(host, 4.0, 3)
    assert status == 0 and route(3) == [DIRECT] * 3
    want = [m.to_host() for m in want]
    groups(spread=True)                                          # exchange through memory: the same sums
    msgs, per, status, _ = encode(host, 4.0, 3)
    assert status == 0 and route(3) == [DIRECT] * 3
    for a, m in zip(want, msgs):
        b = m.to_host()
        assert all(np.array_equal(a[k], b[k]) for k in ("idx", "w", "U", "V"))
    for spread in (False, True):
        groups(spread=spread, start_ticks=0)                     # every workgroup gives up: one reduces the matrix
        msgs, per, status, _ = encode(host, 4.0, 3)
        assert status == 0 and route(3) == [DIRECT] * 3
        for j, (G, msg, (sigma, p)) in enumerate(zip(host, msgs, per)):
            full_parity(G, 4.0, 3, j, msg, sigma, p)
    groups()
    msgs, _, status, _ = encode(host, 4.0, 3)
    assert status == 0 and all(np.array_equal(a[k], m.to_host()[k]) for a, m in zip(want, msgs) for k in ("idx", "w", "U", "V"))


@pytest.mark.parametrize("shape", [(40, 90), (300, 400), (310, 260), (600, 640)])
@pytest.mark.parametrize("kind", ["equal", "tail"])
@pytest.mark.parametrize("folded", [False, True])
def test_a_matrix_that_falls_short_with_nothing_behind_it_still_has_an_unbiased_message(shape, kind, folded):
    # vectors that were not accepted stayed in the message, several of them the same one
    rng = np.random.default_rng(shape[0])
    r = min(shape)
    easy = inputs.low_rank_plus_noise(rng, *shape, [1.0, 0.5], 0.05)
    G = np.zeros(shape, dtype=np.float32)
    if kind == "equal":                                          # every singular value is 2
        np.fill_diagonal(G, 2.0)
    else:
        G = nearly_equal_tail(rng, *shape, 1e-2)
    c = binding.Context(0)
    sigma, p = torch.zeros(r, device="cuda"), torch.zeros(r, device="cuda")
    msg = [binding.alloc_svd_message(*shape, r, "cuda", folded=folded)]
    for g, want in ((easy, 0), (easy, 0), (G, binding.ATOMO_ENOCONV)):
        binding.atomo_encode_svd(c, [dev(g)], 20.0, 3, 8, msgs=msg, sigma_out=sigma, p_out=p, adaptive=1)
        assert c.status()[0] == want
    h = msg[0].to_host()
    A = (G if shape[0] <= shape[1] else G.T).astype(np.float64)
    norms = np.linalg.norm(A, axis=1)
    p = p.cpu().numpy()
    np.testing.assert_allclose(sigma.cpu().numpy(), np.sort(norms)[::-1], rtol=1e-6)
    np.testing.assert_allclose(p, oracle.probabilities(np.sort(norms)[::-1], 20.0), rtol=1e-5)
    assert np.array_equal(h["idx"], np.flatnonzero(oracle.bernoulli_mask(p, 3, 8))) and h["count"] > 5
    dense = binding.atomo_decode(c, msg).cpu().numpy()
    rows = dense if shape[0] <= shape[1] else dense.T
    kept = np.flatnonzero(np.linalg.norm(rows, axis=1))          # whole vectors, each over its probability
    assert kept.size == h["count"]
    np.testing.assert_allclose(np.sort(np.linalg.norm(rows[kept], axis=1)), np.sort(sigma.cpu().numpy()[h["idx"]] / p[h["idx"]]), rtol=1e-5)
    scale = np.linalg.norm(rows[kept], axis=1) / norms[kept]
    assert np.abs(rows[kept] - A[kept] * scale[:, None]).max() <= 1e-5 * np.abs(rows).max()
    binding.atomo_encode_svd(c, [dev(G)], 20.0, 3, 8, msgs=msg, adaptive=1)
    assert c.status()[0] == 0                                    # the next call has the iteration


def test_a_set_whose_iteration_fits_the_address_range_is_accepted_whatever_the_direct_encode_takes():
    # work items of the iteration address 64 GiB of workspace; the direct encode's part (another 44 GB here) is not among that
    n, shape = 2800, (640, 640)
    if torch.cuda.mem_get_info()[0] < 120 << 30:
        pytest.skip("needs 120 GB of free device memory")
    c = binding.Context(0)
    G = dev(inputs.low_rank_plus_noise(np.random.default_rng(0), 640, 640, [1.0, 0.5], 0.02))
    msgs = [binding.alloc_svd_message(*shape, 8, "cuda") for _ in range(n)]
    binding.atomo_encode_svd(c, [G] * n, 2.0, 1, msgs=msgs, stream_ids=[5 + j % 7 for j in range(n)])
    assert c.status()[0] == 0
    one = binding.Context(0)
    for j in (0, 1, 1150, n - 1):
        want = binding.atomo_encode_svd(one, [G], 2.0, 1, stream_ids=[5 + j % 7])[0].to_host()
        got = msgs[j].to_host()
        assert one.status()[0] == 0 and all(np.array_equal(want[k], got[k]) for k in ("idx", "w", "U", "V"))
    c.close()


@pytest.mark.parametrize("r", [33, 64, 128, 129])
@pytest.mark.parametrize("M", [129, 320, 321, 385, 4099])
@pytest.mark.parametrize("tall", [False, True])
def test_sizes_around_the_partial_sums_of_a_gram_product(r, M, tall):
    """Matrices of up to three tiles are cut into chunks of 64 columns, others of 128, and five partial tiles are added up at a time."""
    rng = np.random.default_rng(r + M)
    m, n = (M, r) if tall else (r, M)
    G = inputs.low_rank_plus_noise(rng, m, n, [1.0, 0.5, 0.25, 0.1], 0.02)
    msgs, per, status, _ = encode([G], 3.0, 5, stream_base=r, capacity=r)
    assert status == 0
    full_parity(G, 3.0, 5, r, msgs[0], *per[0])


OF_EIGHT = {
    "up to 384 rows": [(129, 140), (130, 300), (256, 300), (257, 258), (320, 400), (383, 390), (384, 500)] * 3,
    "beside larger ones": [(385, 400), (512, 520), (640, 650)] + [(129, 131), (200, 260), (320, 330), (384, 390)] * 4 + [(64, 80), (128, 140)] * 3,
    "behind larger groups": [(385, 390), (449, 460), (512, 520), (513, 520), (640, 650)] * 5 + [(250, 260), (384, 390), (100, 130), (40, 60)],
}


@pytest.mark.parametrize("kind", OF_EIGHT)
def test_groups_of_eight_workgroups_give_the_bits_of_larger_ones(groups, kind):
    shapes = OF_EIGHT[kind]
    n = len(shapes)
    first = {s: j for j, s in reversed(list(enumerate(shapes)))}
    host = [inputs.low_rank_plus_noise(np.random.default_rng(j % 2), *s, [1.0, 0.5, 0.2], 0.02) for j, s in enumerate(shapes)]
    host[1][5:9] = 0                                             # (a few rows of zeros)
    mats = [dev(g) for g in host]

    def check(msgs, wanted):
        assert ctx().status()[0] == 0 and route(n) == [DIRECT] * n
        for j, want in wanted.items():
            got = msgs[j].to_host()
            assert got["count"] == want["count"] and all(np.array_equal(got[k], want[k]) for k in ("idx", "w", "U", "V")), shapes[j]

    own = {}
    for j in sorted(set(first.values()) | {1, n - 1}):
        own[j] = binding.atomo_encode_svd(ctx(), [mats[j]], 3.0, 6, j)[0].to_host()
    # (nothing that an earlier call left in the workspace counts)
    binding.atomo_encode_svd(ctx(), [torch.full((640, 700), float("nan"), device="cuda")] * n, 3.0, 6, 0)
    assert ctx().status()[0] != 0
    check(binding.atomo_encode_svd(ctx(), mats, 3.0, 6, 0), own)
    groups(spread=True)                                          # exchange through memory
    check(binding.atomo_encode_svd(ctx(), mats, 3.0, 6, 0), own)
    groups(start_ticks=0)                                        # every workgroup gives up: one reduces the matrix
    msgs, per, status, _ = encode(host, 3.0, 6)
    check(msgs, {})
    for j in first.values():
        full_parity(host[j], 3.0, 6, j, msgs[j], *per[j])


@pytest.mark.parametrize("kind", ["pairs", "graded", "even", "one_octave"])
@pytest.mark.parametrize("r", [64, 130, 300])
def test_eigenvalues_that_are_close_to_each_other_or_far_apart(r, kind):
    """Pairs 2e-7 apart, a factor 2^(1/20) from each to the next, even steps, all within one octave; by 32 points per eigenvalue and, in a
    call of many, by 4.  The search ends at 2^-27 of lambda, a float is rounded by 6e-8."""
    rng = np.random.default_rng(r)
    j = np.arange(r)
    sv = {"pairs": 2.0 ** (-(j // 2) / 24.0) * (1.0 - 2e-7 * (j % 2)), "graded": 2.0 ** (-j / 20.0), "even": 1.0 - j / (r + 1.0),
          "one_octave": 1.0 - 0.5 * np.sort(rng.random(r))}[kind]
    u, _ = np.linalg.qr(rng.standard_normal((r, r)))
    v, _ = np.linalg.qr(rng.standard_normal((r + 40, r)))
    G = dev(((u * sv) @ v.T).astype(np.float32))
    want = np.linalg.svd(G.cpu().numpy().astype(np.float64), compute_uv=False)
    got = []
    for n in (1, 70 * 300 // r):
        sigma = torch.zeros(n * r, device="cuda")
        binding.atomo_encode_svd(ctx(), [G] * n, 0.25, 3, 0, sigma_out=sigma)
        assert ctx().status()[0] == 0 and route(n)[0] == DIRECT
        got.append(sigma[:r].cpu().numpy())
        np.testing.assert_allclose(got[-1], want, rtol=1e-7, atol=1e-9 * want[0])
    assert np.array_equal(*got)


@pytest.mark.parametrize("r", [33, 64, 255, 256, 257, 512, 513, 640])
def test_selection_at_the_edges_of_a_thread_s_share(r):
    """One, two and three values per thread, and the last thread's share cut off; budgets that keep nearly nothing and nearly everything
    that has a singular value, equal ones and zeros among them."""
    rng = np.random.default_rng(r)
    G = inputs.low_rank_plus_noise(rng, r, r + 30, [1.0, 0.5, 0.25, 0.1], 0.02)
    dead = G.copy()
    dead[rng.choice(r, r - 24, replace=False)] = 0               # 24 singular values
    for G, s in ((G, 0.01), (G, 5.0), (dead, 2.0), (dead, 24.0)):
        msgs, per, status, _ = encode([G], s, 8, stream_base=1, capacity=r)
        sigma, p = per[0]
        assert status == 0
        p_ref = oracle.probabilities(sigma.astype(np.float64), s)
        np.testing.assert_allclose(p, p_ref, rtol=1e-5, atol=1e-12)
        mask = oracle.bernoulli_mask(p, 8, 1)
        assert np.array_equal(msgs[0].to_host()["idx"], np.flatnonzero(mask))


@pytest.mark.parametrize("shape", [(96, 400), (400, 96), (300, 700), (513, 521)])
@pytest.mark.parametrize("s", [5.0, 8.0, 17.0])
def test_messages_of_more_atoms_than_a_pass_over_the_data_takes(shape, s):
    rng = np.random.default_rng(shape[0])
    G = inputs.low_rank_plus_noise(rng, *shape, [1.0, 0.8, 0.6, 0.5, 0.4, 0.3, 0.25, 0.2], 0.01)
    msgs, per, status, _ = encode([G], s, 11, stream_base=4, capacity=40)
    assert status == 0 and route() == [DIRECT]
    count = msgs[0].to_host()["count"]
    # eight atoms per pass, summed four at a time: a pass with a second sum, a second pass, a third; the last sum of fewer than four
    assert {5.0: 4 < count <= 8, 8.0: 8 < count <= 16, 17.0: 16 < count <= 24}[s] and count % 4 != 0
    full_parity(G, s, 11, 4, msgs[0], *per[0])


def test_a_captured_call_replays_with_its_forks_and_joins():
    """The events of a call that is captured are records of their own, not the completion of its kernels."""
    rng = np.random.default_rng(77)
    shapes = [(64, 27), (130, 700), (10, 512)]
    mats, other = [[dev(inputs.low_rank_plus_noise(rng, m, n, [1.0, 0.5, 0.25], 0.01)) for m, n in shapes] for _ in range(2)]
    c, stream = binding.Context(0), torch.cuda.Stream()
    buffers = [g.clone() for g in mats]
    with torch.cuda.stream(stream):
        msgs = binding.atomo_encode_svd(c, buffers, 3.0, 4, 9)
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=stream, capture_error_mode="relaxed"):
            binding.atomo_encode_svd(c, buffers, 3.0, 4, 9, msgs=msgs)
    for given in (other, mats, other):
        want = binding.atomo_encode_svd(ctx(), given, 3.0, 4, 9)
        for b, g in zip(buffers, given):
            b.copy_(g)
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        for a, b in zip(msgs, want):
            got, ref = a.to_host(), b.to_host()
            assert np.array_equal(got["idx"], ref["idx"]) and np.array_equal(got["w"], ref["w"])
            assert np.array_equal(got["U"], ref["U"]) and np.array_equal(got["V"], ref["V"])


@pytest.mark.parametrize("shape", [(33, 70), (64, 576), (128, 300), (300, 200), (512, 700)])
@pytest.mark.parametrize("apart", [0.1, 1e-3, 1e-5])
def test_vectors_of_neighbours_near_and_far(shape, apart):
    """Kept singular vectors against those of LAPACK.  A vector of an eigenvalue found to 2^-20 of its cell takes one round, a neighbour in
    the way a second one; either way it may turn by 1e-9 (the first round's bound) and by the rounding of the Gram matrix (2e-15 of the
    largest eigenvalue, with `apart` between neighbours), and every entry is rounded to fp32 (6e-8 of the norm)."""
    rng = np.random.default_rng(shape[0] + int(1e6 * apart))
    G = inputs.low_rank_plus_noise(rng, *shape, [1.0, 0.8, 0.8 * (1.0 - apart), 0.5, 0.25], 1e-4)
    msgs, per, status, _ = encode([G], 20.0, 3, stream_base=1, capacity=min(shape))
    assert status == 0 and route() == [DIRECT]
    host = msgs[0].to_host()
    U, S, Vt = np.linalg.svd(np.asarray(G, dtype=np.float64), full_matrices=False)
    kept = [k for k, i in enumerate(host["idx"]) if i < 5]
    assert len(kept) == 5                                        # (p = 1 for all of them)
    for k in kept:
        i = int(host["idx"][k])
        u, v = host["U"][:, k].astype(np.float64), host["V"][:, k].astype(np.float64)
        gap = np.min(np.abs(np.delete(S, i) ** 2 - S[i] ** 2))
        sign = np.sign(u @ U[:, i])
        bound = 1e-9 + 6e-8 + 1e-14 * S[0] ** 2 / gap
        assert np.linalg.norm(sign * u - U[:, i]) < bound
        assert np.linalg.norm(sign * v - Vt[i]) < bound * (1.0 + S[0] / S[i])
