"""GPU parity: entry-wise ATOMO encode / decode against the oracle."""
import numpy as np
import pytest
import torch

import oracle
from paper_1806_04090_amd import binding, inputs
from gpu_common import ctx, dev, uniforms_on_the_device

pytestmark = pytest.mark.gpu


def encode(g, s, seed, stream, capacity=None):
    d = dev(g)
    p = torch.zeros(g.size, dtype=torch.float32, device="cuda")
    msg = None if capacity is None else binding.alloc_entrywise_message(g.size, capacity, "cuda")
    msg = binding.atomo_encode_entrywise(ctx(), d, s, seed, stream, msg=msg, p_out=p)
    status, _ = ctx().status()
    return msg, p.cpu().numpy(), status


def parity(g, s, seed, stream, capacity=None):
    msg, p_gpu, status = encode(g, s, seed, stream, capacity)
    assert status == 0
    p_ref = oracle.probabilities(g.astype(np.float64), s)
    np.testing.assert_allclose(p_gpu, p_ref, rtol=1e-6, atol=1e-12)
    h = msg.to_host()
    ref = oracle.encode_entrywise(g, s, seed, stream, p32=p_gpu)          # oracle chain from the GPU's p
    assert h["count"] == ref["idx"].size
    assert np.array_equal(h["idx"], ref["idx"])                            # bit-exact mask, ascending order
    np.testing.assert_allclose(h["val"], ref["val"], rtol=1e-6)
    # how far the mask moves if the oracle's own p is used instead (reported property: tiny)
    own = oracle.encode_entrywise(g, s, seed, stream)
    assert len(set(own["idx"]) ^ set(h["idx"])) <= max(2, int(1e-4 * max(1, h["count"])))
    return msg, h, p_gpu


@pytest.mark.parametrize("n", [1, 3, 4, 5, 255, 4096, 4097, 10_001, 70_000])
def test_sizes_with_ragged_tails(n):
    g = inputs.flat_heavy_tail(seed=n, n=n, heavy_fraction=0.01)
    s = max(0.5, n / 50)
    parity(g, s, 3, 9)


def test_config2_shape_at_reduced_size_then_decode():
    n = 1_000_003
    g = inputs.flat_heavy_tail(seed=0, n=n)
    msg, h, p = parity(g, n / 100, 0, 0)
    out = binding.atomo_decode(ctx(), [msg]).cpu().numpy()
    want = oracle.decode_entrywise([h], n)
    np.testing.assert_allclose(out, want.astype(np.float32), rtol=1e-6, atol=0)
    assert (out != 0).sum() == h["count"]
    # uncapped kept values all carry the one magnitude tail/(s - n_s)  (eq. (p_i), KKT appendix)
    mags = np.abs(h["val"][p[h["idx"]] < 1])
    assert mags.size > 0 and (mags.max() - mags.min()) <= 1e-6 * mags.max()


def test_unaligned_pointer_and_streams():
    g_full = inputs.flat_heavy_tail(seed=2, n=50_001)
    d = dev(g_full)
    view = d[1:]                                                 # 4-byte aligned only
    g = g_full[1:]
    p = torch.zeros(g.size, dtype=torch.float32, device="cuda")
    msg = binding.atomo_encode_entrywise(ctx(), view, 500.0, 1, 2, p_out=p)
    assert ctx().status()[0] == 0
    ref = oracle.encode_entrywise(g, 500.0, 1, 2, p32=p.cpu().numpy())
    assert np.array_equal(msg.to_host()["idx"], ref["idx"])
    other = binding.atomo_encode_entrywise(ctx(), view, 500.0, 1, 3)
    assert not np.array_equal(other.to_host()["idx"], ref["idx"])


def test_degenerate_inputs():
    zeros = np.zeros(5000, dtype=np.float32)
    msg, p, status = encode(zeros, 10.0, 0, 0)
    assert status == 0 and msg.to_host()["count"] == 0 and (p == 0).all()
    g = inputs.flat_heavy_tail(seed=3, n=3000)
    msg, p, status = encode(g, 5000.0, 0, 0, capacity=3000)      # s >= n: nothing is dropped
    h = msg.to_host()
    assert status == 0 and h["count"] == int((g != 0).sum())
    out = binding.atomo_decode(ctx(), [msg]).cpu().numpy()
    np.testing.assert_array_equal(out, g)
    equal = np.full(9000, 0.25, dtype=np.float32)
    parity(equal, 90.0, 4, 4)


def test_capacity_overflow_is_latched():
    g = inputs.flat_heavy_tail(seed=4, n=20_000)
    msg, p, status = encode(g, 2000.0, 0, 0, capacity=100)
    assert status == binding.ATOMO_ECAPACITY
    h = msg.to_host()
    full = oracle.encode_entrywise(g, 2000.0, 0, 0, p32=p)
    assert h["count"] == full["idx"].size and np.array_equal(h["idx"], full["idx"][:100])


def test_determinism_and_multi_message_average():
    g = inputs.flat_heavy_tail(seed=5, n=200_000)
    a = binding.atomo_encode_entrywise(ctx(), dev(g), 2000.0, 8, 0).to_host()
    b = binding.atomo_encode_entrywise(ctx(), dev(g), 2000.0, 8, 0).to_host()
    assert np.array_equal(a["idx"], b["idx"]) and np.array_equal(a["val"], b["val"])
    msgs = [binding.atomo_encode_entrywise(ctx(), dev(g), 2000.0, 8, w) for w in range(4)]
    out = binding.atomo_decode(ctx(), msgs, scale=0.25).cpu().numpy()
    want = oracle.decode_entrywise([m.to_host() for m in msgs], g.size, scale=0.25)
    np.testing.assert_allclose(out, want, rtol=1e-5, atol=1e-9)
    # overlapping messages are added in call order, one launch each: the same bits in every run
    for _ in range(3):
        again = binding.atomo_decode(ctx(), msgs, scale=0.25).cpu().numpy()
        assert np.array_equal(out, again)
    assert (np.count_nonzero(sum((np.bincount(m.to_host()["idx"], minlength=g.size) for m in msgs))) <
            sum(m.to_host()["count"] for m in msgs))            # the messages do overlap


def test_unbiased_over_streams():
    g = inputs.flat_heavy_tail(seed=6, n=2000, heavy_fraction=0.01)
    trials = 300
    acc = np.zeros(g.size); acc2 = np.zeros(g.size)
    d = dev(g)
    for t in range(trials):
        out = binding.atomo_decode(ctx(), [binding.atomo_encode_entrywise(ctx(), d, 100.0, 21, t)]).cpu().numpy().astype(np.float64)
        acc += out; acc2 += out * out
    mean = acc / trials
    var = acc2 / trials - mean ** 2
    # z-test where the normal approximation holds (enough expected hits); exact where p = 1
    p = oracle.probabilities(g.astype(np.float64), 100.0)
    often = (p * trials >= 30) & (p < 1)
    assert often.sum() > 20
    z = (mean[often] - g[often]) / np.sqrt(g[often].astype(np.float64) ** 2 * (1 - p[often]) / p[often] / trials)
    assert np.abs(z).max() < 5.0
    np.testing.assert_array_equal(mean[p == 1], g[p == 1].astype(np.float64))
    # and the whole vector: sum of the estimates against the sum of the gradient
    total_var = (g.astype(np.float64) ** 2 * (1 - p) / np.maximum(p, 1e-300))[p > 0].sum() / trials
    assert abs(mean.sum() - g.astype(np.float64).sum()) < 5 * np.sqrt(total_var)


def test_largest_supported_length():
    # n just below 2^32 (17 GB of gradient, generated on the device): no oracle pass over that, so the properties
    # that hold at any size: kept count within 6 sd of s, ascending indices past 2^31, capped entries unchanged
    # (p = 1), every other kept value of the one magnitude tail / (s - n_s) (eq. (p_i), KKT appendix), which is
    # also evaluated directly; decode puts the values where they belong and zeros elsewhere
    n = 2 ** 32 - 4099
    gen = torch.Generator(device="cuda")
    gen.manual_seed(1)
    g = torch.empty(n, dtype=torch.float32, device="cuda")
    step = 1 << 28
    for a in range(0, n, step):
        g[a:min(n, a + step)].normal_(0.0, 1e-3, generator=gen)
    g[-1] = 7.0
    g[2 ** 31 + 5] = -9.0
    g[0] = 3.0
    s = n / 1000.0
    msg = binding.alloc_entrywise_message(n, int(s + 10 * np.sqrt(s) + 64), "cuda")
    binding.atomo_encode_entrywise(ctx(), g, s, 5, 9, msg=msg)
    assert ctx().status()[0] == 0
    k = int(msg.count.item())
    assert abs(k - s) < 6 * np.sqrt(s)
    idx = msg.idx[:k].to(torch.int64) & 0xFFFFFFFF
    val = msg.val[:k]
    assert bool((idx[1:] > idx[:-1]).all()) and 0 <= int(idx[0]) and int(idx[-1]) < n
    gv = g[idx]
    assert bool((torch.sign(gv) == torch.sign(val)).all())
    capped = val.abs() > 1.0
    assert sorted(idx[capped].tolist()) == [0, 2 ** 31 + 5, n - 1] and torch.equal(val[capped], gv[capped])
    tau = val.abs()[~capped]
    assert float(tau.max() - tau.min()) <= 2e-6 * float(tau.max())
    l1 = sum(float(g[a:min(n, a + step)].abs().double().sum()) for a in range(0, n, step))
    assert abs(float(tau.max()) - (l1 - 19.0) / (s - 3)) <= 1e-5 * float(tau.max())
    del gv
    out = binding.atomo_decode(ctx(), [msg])
    assert torch.equal(out[idx], val)
    total = sum(float(out[a:min(n, a + step)].abs().double().sum()) for a in range(0, n, step))
    assert abs(total - float(val.abs().double().sum())) <= 1e-9 * total
    del out, g
    torch.cuda.empty_cache()


@pytest.mark.parametrize("kind", ["dense", "dense_here_and_there", "subnormal", "subnormal_dense", "subnormal_wide", "last_bucket"])
@pytest.mark.parametrize("n", [17_000, 300_001, 4_200_003])
def test_records_that_the_second_search_level_leaves_open(kind, n):
    """Open records in segments with and without slots for all candidates; more of them than the list holds (all nonzero elements
    where a bucket reaches down to zero, one draw in 170 at a level of 2.4e-40); the water level in the last bucket of its level, at 1.12494 = 1.125 - 2^-14.02."""
    rng = np.random.default_rng(n)
    g = (rng.standard_normal(n) * 0.5).astype(np.float32)
    s = 0.3 * n
    if kind == "dense_here_and_there":
        g[rng.random(n) < np.where(np.arange(n) // 5000 % 2, 0.0, 0.97)] = 0
        s = 0.2 * n
    elif kind.startswith("subnormal"):
        g = (rng.integers(-200, 201, n) * 2.0 ** -149).astype(np.float32)
        s = 0.4 * n
        if kind == "subnormal":                                  # (slots for them all)
            g[rng.random(n) < 0.95] = 0
            s = n / 100
        elif kind == "subnormal_wide":
            g, s = rng.uniform(0.0, 4.0e-40, n).astype(np.float32), 0.7 * n
    elif kind == "last_bucket":
        g = rng.uniform(0.1, 1.0, n).astype(np.float32)
        s = float(g.astype(np.float64).sum()) / 1.12494
    if not kind.startswith("subnormal"):
        parity(g, s, 5, 2, capacity=n)
        return
    msg, p, status = encode(g, s, 5, 2, capacity=n)
    np.testing.assert_allclose(p, oracle.probabilities(g.astype(np.float64), s), rtol=1e-6, atol=1e-12)
    h, ref = msg.to_host(), oracle.encode_entrywise(g, s, 5, 2, p32=p)
    assert status == 0 and np.array_equal(h["idx"], ref["idx"])
    np.testing.assert_allclose(h["val"], ref["val"], rtol=1e-6, atol=2.0 ** -149)        # (a value is rounded to a multiple of that)


@pytest.fixture
def counts():
    yield ctx().debug_entrywise_counts
    ctx().debug_entrywise_counts()


@pytest.mark.parametrize("n", [16_385, 70_000, 300_001])
def test_counts_of_other_workgroups_that_do_not_come(counts, n):
    # 5, 18 and 74 groups, the last of one segment (a wave looks for 64 counts at a time); looked for once, and not at all
    g = (np.random.default_rng(n).integers(-200, 201, n) * 2.0 ** -149).astype(np.float32)
    msg, p, status = encode(g, 0.4 * n, 5, 2, capacity=n)
    h = msg.to_host()
    assert status == 0 and np.array_equal(h["idx"], oracle.encode_entrywise(g, 0.4 * n, 5, 2, p32=p)["idx"])
    for loads in (1, 0):
        counts(loads)
        msg, _, status = encode(g, 0.4 * n, 5, 2, capacity=n)
        again = msg.to_host()
        assert status == 0 and again["count"] == h["count"] and all(np.array_equal(again[k], h[k]) for k in ("idx", "val"))


@pytest.mark.parametrize("kind", ["slots", "dense"])                       # segments with and without slots for their candidates
@pytest.mark.parametrize("level", [5.0e-32, 6.0e-32, 9.7e-32, 1.2e-31])
def test_water_levels_where_the_scaled_ratio_leaves_the_float_range(level, kind):
    # 2^24 / level against the largest float, 3.4e38: the single-precision bounds of p change their form at a level of 1e-31
    n = 100_001 if kind == "slots" else 2_000_003
    rng = np.random.default_rng(7)
    g = rng.standard_normal(n)
    if kind == "slots":                                                   # (behind the level's last bound every nonzero is a candidate)
        g[rng.random(n) < 0.95] = 0
    s = n / 100 if kind == "slots" else 0.3 * n
    p = oracle.probabilities(g, s)
    g = (g * (level * np.max(p[g != 0] / np.abs(g[g != 0])))).astype(np.float32)          # (an uncapped p is |g| / level)
    p_gpu = parity(g, s, 21, 4)[2]
    free = (p_gpu > 0) & (p_gpu < 1)
    np.testing.assert_allclose(np.abs(g[free]) / p_gpu[free], level, rtol=1e-5)


@pytest.mark.parametrize("kind", ["dense", "slots"])
@pytest.mark.parametrize("x", [2.0 ** -149, 2.0 ** -143, 2.0 ** -142, 2.0 ** -137, 2.0 ** -101])
def test_a_draw_of_zero_against_a_probability_below_the_normal_range(x, kind):
    # element 227537 draws 0 and is kept if its p is more than 0 as a float: the smallest is 2^-149, p = x / level
    n, at = 300_001, 227_537
    assert oracle.uniforms(58, 2, n)[at] == 0
    rng = np.random.default_rng(0)
    g = (rng.standard_normal(n) * 50).astype(np.float32)
    if kind == "slots":
        g[rng.random(n) < 0.95] = 0
    g[at] = x
    _, h, p_gpu = parity(g, 0.3 * n if kind == "dense" else n / 100, 58, 2, capacity=n)
    level = 132.7 if kind == "dense" else 202.9
    assert (at in h["idx"]) == (x / level > 2.0 ** -150) == (p_gpu[at] > 0)


@pytest.mark.parametrize("n, seed, at", [(16_000, 1246, 10_044), (300_001, 58, 227_537)])
def test_a_draw_of_zero_below_a_water_level_beyond_the_float_range(n, seed, at):
    # a budget so small that 2^24 / level is zero as a float: the one element that draws 0 has p = 1e-19 to 1e-18 and is kept
    # (with a value of the level, which no float holds)
    assert list(np.flatnonzero(oracle.uniforms(seed, 2, n) == 0)) == [at]
    g = (np.random.default_rng(n).uniform(0.5e38, 1e38, n)).astype(np.float32)
    msg, p, status = encode(g, 1e-13, seed, 2, capacity=8)
    np.testing.assert_allclose(p, oracle.probabilities(g.astype(np.float64), 1e-13), rtol=1e-6)
    h = msg.to_host()
    assert status == 0 and list(h["idx"]) == [at] and np.isinf(h["val"][0])


@pytest.mark.parametrize("kind", ["multiples", "wide"])
def test_a_subnormal_gradient_takes_about_as_long_as_another(kind):
    # one more pass over the gradient, where each workgroup once drew all groups before its own: 12.8 ms instead of 0.2
    n, times = 16_000_001, []
    gen = torch.Generator(device="cuda")
    gen.manual_seed(1)
    normal = torch.randn(n, generator=gen, device="cuda")
    if kind == "multiples":
        small, s = torch.randint(-200, 201, (n,), generator=gen, device="cuda").float() * 2.0 ** -149, 0.4 * n
    else:
        small, s = torch.rand(n, generator=gen, device="cuda") * 4.0e-40, 0.7 * n
    msg = binding.alloc_entrywise_message(n, n, "cuda")
    for g in (normal, small):
        took = []
        for _ in range(5):
            start, end = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            start.record()
            binding.atomo_encode_entrywise(ctx(), g, s, 5, 2, msg=msg)
            end.record()
            end.synchronize()
            took.append(start.elapsed_time(end))
        times.append(min(took))
    assert ctx().status()[0] == 0
    assert times[1] < 6 * times[0], times


def encode_time(g, s, msg, seed=5, calls=1):
    """Least time of seven encodes (or times `calls` of them), in milliseconds."""
    took = []
    for _ in range(7):
        start, end = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        start.record()
        for _ in range(calls):
            binding.atomo_encode_entrywise(ctx(), g, s, seed, 2, msg=msg)
        end.record()
        end.synchronize()
        took.append(start.elapsed_time(end))
    return min(took)


@pytest.mark.parametrize("n", [16_000_001, 2 ** 25 + 5])
@pytest.mark.parametrize("down", [92, 94, 96, 98])
def test_a_tiny_water_level_takes_about_as_long_as_another(n, down):
    """Levels of 2^-96.6 to 2^-102.6, where 2^32 over the level does not fit a float but 2^24 over it does, zeros among the elements: the
    same draws are kept, with values smaller by just that power, and no more elements are looked at (but a long gradient is read twice, as
    one whose level no sample predicts)."""
    gen = torch.Generator(device="cuda")
    gen.manual_seed(3)
    g = torch.randn(n, generator=gen, device="cuda") * 1e-3
    g[torch.randint(0, n, (n // 1000,), generator=gen, device="cuda")] *= 100
    g[torch.rand(n, generator=gen, device="cuda") < 0.5] = 0
    small = g * 2.0 ** -down
    msgs = [binding.alloc_entrywise_message(n, n, "cuda") for _ in range(2)]
    times = [encode_time(x, 0.01 * n, m) for x, m in zip((g, small), msgs)]
    assert ctx().status()[0] == 0
    a, b = (m.to_host() for m in msgs)
    assert a["count"] == b["count"] > 0.009 * n and np.array_equal(a["idx"], b["idx"])
    assert np.array_equal(a["val"], b["val"].astype(np.float64) * 2.0 ** down)
    assert times[1] < (1.5 if n < 2 ** 25 else 2.2) * times[0], times


@pytest.mark.parametrize("seed", [1, 2])
def test_the_sum_below_a_sampled_window_is_good_to_the_last_bit(seed):
    """All elements lie below the level, from 1 down to 2^-30, and the budget is such that p of the largest one is rounded one way with their sum
    rounded once and the other way with a sum that is one unit of 2^-53 larger (or smaller: the second budget).  Added up as one number
    over the workgroups the sum of seed 1 is one unit too large, that of seed 2 one too small."""
    n = 2 ** 25
    g = np.exp2(np.random.default_rng(seed).uniform(-30, 0, n)).astype(np.float32)
    at, total = int(np.argmax(g)), float(g.astype(np.longdouble).sum())
    a = float(g[at])
    for other in (np.nextafter(total, np.inf), np.nextafter(total, 0.0)):
        p, s = np.float32(a * 1000.0 / total), 0.0
        while not s:
            p = np.nextafter(p, np.float32(1.0))
            tie = (float(p) + float(np.nextafter(p, np.float32(1.0)))) / 2
            tries = tie * total / a + np.arange(-8, 9) * np.spacing(1000.0)
            rounded = [(tries / x * a).astype(np.float32) for x in (total, other)]
            s = next(iter(tries[rounded[0] != rounded[1]]), 0.0)
        want = np.float32(s / total * a)
        _, p_gpu, status = encode(g, float(s), 5, 2, capacity=4000)
        assert status == 0 and p_gpu[at] == want


PIECE, PIECES = 32, 2 ** 15


def sampled(n):
    """Mask of the elements that the sample of a long gradient reads: PIECE of them at a hashed place of each of PIECES parts."""
    piece, spacing = np.arange(PIECES, dtype=np.uint64), n // PIECES // PIECE
    m32 = np.uint64(0xFFFFFFFF)
    h = ((piece * np.uint64(0x9E3779B1)) & m32) ^ (((piece * np.uint64(0x85EBCA6B)) & m32) >> np.uint64(15))
    at = (piece * np.uint64(spacing) + ((h * np.uint64(spacing)) >> np.uint64(32))) * np.uint64(PIECE)
    mask = np.zeros(n, dtype=bool)
    mask[(at[:, None] + np.arange(PIECE, dtype=np.uint64)).astype(np.int64)] = True
    return mask


def alike_neighbours(rng, n, length, active, noise):
    """Rows of `length` elements, a share of them `active` with scales of their own, the others `noise` times as large."""
    rows = -(-n // length)
    g = rng.standard_normal((rows, length), dtype=np.float32)
    on = rng.random(rows) < active
    g *= ((on + noise) * np.exp(0.5 * rng.standard_normal(rows)) * 1e-3).astype(np.float32)[:, None]
    return g.ravel()[:n]


@pytest.mark.parametrize("length, active, noise, keep, seed", [(64, 0.03, 0.0, 0.01, 0), (64, 0.02, 0.0, 0.001, 2), (64, 0.02, 1e-2, 0.01, 2),
                                                               (512, 0.02, 0.0, 0.001, 0)])
def test_a_long_gradient_whose_neighbours_are_alike_is_read_once(length, active, noise, keep, seed):
    """Inputs at which 16384 pieces of 64, taken for 2^20 independent elements, were sure of a level that is 6 to 12 % off, or would say
    that they cannot tell.  Those were read two and three times: 1.7 to 2.4 times as long."""
    n = 2 ** 25
    g = alike_neighbours(np.random.default_rng(seed), n, length, active, noise)
    plain = np.random.default_rng(seed).standard_normal(n, dtype=np.float32)
    msg = binding.alloc_entrywise_message(n, n // 10, "cuda")
    time_plain = encode_time(dev(plain), keep * n, msg)
    time = encode_time(dev(g), keep * n, msg)
    _, h, _ = parity(g, keep * n, 5, 2, capacity=n // 10)
    got = msg.to_host()
    assert h["count"] == got["count"] and np.array_equal(h["idx"], got["idx"]) and np.array_equal(h["val"], got["val"])
    assert time < 1.5 * time_plain, (time, time_plain)


@pytest.mark.parametrize("length, active", [(64, 0.005), (64, 0.012)])
def test_a_long_gradient_of_zeros_takes_no_longer_for_a_sample_that_cannot_say(length, active):
    """Fewer elements that are not zero than the budget, or about as many: no sample finds a level, and level 0 is formed of all elements,
    most of them in one bucket.  Twice the time of a gradient without zeros where those are counted, one by one; less without."""
    n = 2 ** 25 + 1
    g = alike_neighbours(np.random.default_rng(7), n, length, active, 0.0)
    plain = np.random.default_rng(7).standard_normal(n, dtype=np.float32)
    msg = binding.alloc_entrywise_message(n, n // 10, "cuda")
    time_plain = encode_time(dev(plain), n / 100, msg)
    time = encode_time(dev(g), n / 100, msg)
    parity(g, n / 100, 5, 2, capacity=n // 10)
    assert time < 1.6 * time_plain, (time, time_plain)


@pytest.mark.parametrize("kind, extra", [("heavy", 0), ("heavy", 4099), ("all_alike", 3), ("many_near_the_level", 1), ("above_the_window", 2),
                                         ("below_the_window", 5), ("scattered", 1), ("zeros", 7), ("subnormal", 0), ("everything", 0)])
def test_long_gradients_whose_level_a_sample_predicts(kind, extra):
    """From 2^25 elements on.  The level is where the sample says, with few values near it or so many that they go through LDS; it is not,
    because the sample saw none of the large values or nothing but them; the sample cannot say."""
    n = 2 ** 25 + extra
    rng = np.random.default_rng(n)
    g = rng.standard_normal(n, dtype=np.float32) * np.float32(1e-3)
    s = n / 100
    if kind == "heavy":
        g[rng.integers(0, n, n // 1000)] *= 100
    elif kind == "all_alike":                                    # (every p is 0.4, one value)
        g = np.where(rng.random(n, dtype=np.float32) < 0.5, np.float32(0.7), np.float32(-0.7))
        s = 0.4 * n
    elif kind == "many_near_the_level":                          # (and no segment has slots for them)
        s = 0.6 * n
    elif kind == "above_the_window":
        g[~sampled(n)] *= 3
    elif kind == "below_the_window":
        g[sampled(n)] *= 3
    elif kind == "scattered":                                    # (a handful of values holds the budget)
        g[rng.integers(0, n, 40)] = 50.0
        s = 37.5
    elif kind == "zeros":
        g[:] = 0
    elif kind == "subnormal":
        g = (rng.integers(-200, 201, n) * 2.0 ** -149).astype(np.float32)
        g[rng.random(n, dtype=np.float32) < 0.95] = 0
    elif kind == "everything":
        s = 2.0 * n
    d = torch.zeros(n + 4, device="cuda")[extra & 3:][:n]        # (aligned to 4, 8 and 16 bytes)
    d.copy_(torch.from_numpy(g))
    p = torch.zeros(n, device="cuda")
    msg = binding.alloc_entrywise_message(n, n, "cuda")
    for _ in range(2):                                           # (the second call finds what the first one left)
        binding.atomo_encode_entrywise(ctx(), d, s, 5, 2, msg=msg, p_out=p)
    assert ctx().status()[0] == 0
    p = p.cpu().numpy()
    np.testing.assert_allclose(p, oracle.probabilities(g.astype(np.float64), s), rtol=1e-6, atol=1e-12)
    h, ref = msg.to_host(), oracle.encode_entrywise(g, s, 5, 2, p32=p)
    assert h["count"] == ref["idx"].size and np.array_equal(h["idx"], ref["idx"])
    np.testing.assert_allclose(h["val"], ref["val"], rtol=1e-6, atol=2.0 ** -149)


@pytest.mark.parametrize("kind", ["plain", "apart", "scattered", "misleading", "many_near_the_level", "zeros"])
@pytest.mark.parametrize("n", [2 ** 26 + 4099, 2 ** 28 + 3])
def test_longer_gradients_than_one_round_of_the_draws(n, kind):
    """From 2^26 elements on a workgroup of the draws takes several groups of segments, one after the other.  Against torch on the device: p
    is min(1, |g| (s - n_s) / tail), one rounding to fp32 of a value in double precision, with the n_s and the tail that it leaves itself,
    and what is kept is the comparison of the oracle's uniforms with it."""
    gen = torch.Generator(device="cuda")
    gen.manual_seed(n)
    g = torch.randn(n, generator=gen, device="cuda")
    s = n / 100
    if kind == "apart":                                          # (a window of wider buckets: rows that are alike)
        rows = (torch.rand(n // 64 + 1, generator=gen, device="cuda") < 0.03).float() * torch.rand(n // 64 + 1, generator=gen, device="cuda")
        g *= rows.repeat_interleave(64)[:n]
        s = n / 500
    elif kind == "scattered":                                    # (no window)
        g[torch.randint(0, n, (3,), generator=gen, device="cuda")] = float(n)
        s = 2.5
    elif kind == "misleading":                                   # (the level is not in the window)
        g[~torch.from_numpy(sampled(n)).cuda()] *= 3.0
    elif kind == "many_near_the_level":
        s = 0.6 * n
    elif kind == "zeros":
        g[torch.rand(n, generator=gen, device="cuda") < 0.995] = 0
    p = torch.zeros(n, device="cuda")
    msg = binding.alloc_entrywise_message(n, n if s > n / 10 else n // 50, "cuda")
    for _ in range(2):                                           # (the second call finds what the first one left)
        binding.atomo_encode_entrywise(ctx(), g, s, 5, 2, msg=msg, p_out=p)
    assert ctx().status()[0] == 0
    capped = p == 1.0
    tail, n_s, most = 0.0, int(capped.sum()), 0.0
    for part, c in zip(g.split(2 ** 26), capped.split(2 ** 26)):  # (in double precision a part at a time)
        rest = torch.where(c, 0.0, part.abs()).double()
        tail, most = tail + float(rest.sum()), max(most, float(rest.max()))
    ratio = (s - n_s) / tail if tail > 0 else float("inf")
    assert s >= n_s and (tail == 0 or most * ratio <= 1.0 + 2.0 ** -24)
    for part, q in zip(g.split(2 ** 26), p.split(2 ** 26)):
        want = torch.where(part == 0, 0.0, (part.double().abs() * ratio).clamp(max=1.0))
        assert bool(((q.double() - want).abs() <= 2.0 ** -24 * 1.001 * want + 2.0 ** -149).all())
    kept = torch.cat([torch.nonzero(u * 2.0 ** -24 < q).view(-1) + at * 2 ** 26 for at, (u, q) in
                      enumerate(zip(uniforms_on_the_device(n, 2, 5).split(2 ** 26), p.split(2 ** 26)))])
    assert int(msg.count) == kept.numel() > 0
    assert torch.equal(msg.idx[:kept.numel()].long() & 0xFFFFFFFF, kept)
    assert torch.equal(msg.val[:kept.numel()], g[kept] / p[kept])


@pytest.mark.parametrize("kind, keep", [("normal", 0.01), ("normal", 0.3), ("normal", 0.7), ("normal", 1.0), ("two_values", 0.3), ("two_values", 0.7)])
def test_long_and_short_segments_give_one_message(kind, keep):
    """A gradient one element below 2^25, and the same with two zeros behind it, which takes the path of a sample: level, draws and so the message
    are the same, and it takes no longer if its segments run over their slots (the whole gradient kept: 1.37 times as long where a segment
    that had run over went on to queue its candidates)."""
    n = 2 ** 25 - 1
    gen = torch.Generator(device="cuda")
    gen.manual_seed(1)
    g = torch.zeros(n + 2, device="cuda")
    if kind == "normal":
        g[:n].normal_(generator=gen)
    else:
        g[:n] = torch.where(torch.rand(n, generator=gen, device="cuda") < 0.5, 1.0, -1.25)
    msgs = [binding.alloc_entrywise_message(n + k, n, "cuda") for k in (0, 2)]
    times = [encode_time(g[:n + k], keep * n, m) for k, m in zip((0, 2), msgs)]
    assert ctx().status()[0] == 0
    count = int(msgs[0].count)
    assert count == int(msgs[1].count) > 0
    assert torch.equal(msgs[0].idx[:count], msgs[1].idx[:count]) and torch.equal(msgs[0].val[:count], msgs[1].val[:count])
    if keep > 0.01:
        assert times[1] < 1.2 * times[0], times


@pytest.mark.parametrize("kind", ["sparse", "one_magnitude", "unaligned"])
def test_gradients_of_few_buckets_take_no_longer_than_others(kind):
    """Three million elements on 91 workgroups: zeros and equal magnitudes once queued in a few words of each workgroup's LDS (1.4 and 1.3
    times as long as a normal gradient), and one that is not aligned was read an element at a time (1.16 times)."""
    n = 3_000_000
    gen = torch.Generator(device="cuda")
    gen.manual_seed(9)
    g = torch.randn(n + 1, generator=gen, device="cuda")
    if kind == "sparse":
        other = g[:n] * (torch.rand(n, generator=gen, device="cuda") < 0.005)
    elif kind == "one_magnitude":
        other = torch.where(g[:n] > 0, 0.7, -0.7)
    else:
        other = g[1:]
    msgs = [binding.alloc_entrywise_message(n, n, "cuda") for _ in range(2)]
    times = [encode_time(x, n / 100, m, calls=20) for x, m in zip((g[:n], other), msgs)]
    assert times[1] < (1.1 if kind == "unaligned" else 1.2) * times[0], times
    _, h, _ = parity(other.cpu().numpy(), n / 100, 5, 2, capacity=n // 10)
    got = msgs[1].to_host()
    assert h["count"] == got["count"] and np.array_equal(h["idx"], got["idx"]) and np.array_equal(h["val"], got["val"])


@pytest.mark.parametrize("n, offset", [(20_003, 0), (20_003, 1), (60_001, 2), (1_000_002, 3)])
def test_four_neighbours_of_one_bucket_are_counted_together(n, offset):
    """Runs of equal values, of values that share a bucket and of zeros, of lengths that are no multiples of four."""
    rng = np.random.default_rng(n + offset)
    runs = rng.integers(1, 11, n)
    values = np.exp2(rng.integers(-6, 3, n)).astype(np.float32) * rng.choice([0.0, 1.0, -1.0, 1.0], n).astype(np.float32)
    g = np.repeat(values, runs)[:n]
    g *= np.where(rng.random(n) < 0.5, 1.0, 1.0 + rng.random(n) / 20).astype(np.float32)
    flat = torch.zeros(n + 8, device="cuda")
    d = flat[offset:offset + n]
    d.copy_(torch.from_numpy(g))
    for s in (n / 100, n / 5, 0.9 * np.count_nonzero(g), 2.0 * n):
        p = torch.zeros(n, device="cuda")
        msg = binding.atomo_encode_entrywise(ctx(), d, s, 7, 1, msg=binding.alloc_entrywise_message(n, n, "cuda"), p_out=p)
        q = binding.atomo_probabilities(ctx(), d.abs(), [0, n], s)
        assert ctx().status()[0] == 0 and torch.equal(p, q)
        p = p.cpu().numpy()
        np.testing.assert_allclose(p, oracle.probabilities(g.astype(np.float64), s), rtol=1e-6, atol=1e-12)
        h, ref = msg.to_host(), oracle.encode_entrywise(g, s, 7, 1, p32=p)
        assert h["count"] == ref["idx"].size and np.array_equal(h["idx"], ref["idx"])
