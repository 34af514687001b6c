"""GPU parity of the one-launch decode of entry-wise and l_q messages (decode_sparse) at the sizes where it can go wrong:
tile edges, a ragged last tile, unaligned outputs, tiles with more pairs than a group requests at once, runs of several
tiles per workgroup, and more messages than one launch takes."""
import numpy as np
import pytest
import torch

import oracle
from paper_1806_04090_amd import binding
from gpu_common import ctx, dev

pytestmark = pytest.mark.gpu


def entrywise(rng, n, k):
    idx = np.sort(rng.choice(n, size=k, replace=False)) if k < n else np.arange(n)
    val = rng.standard_normal(k).astype(np.float32)
    m = binding.alloc_entrywise_message(n, max(k, 1), "cuda")
    m.count.fill_(k)
    if k:
        m.idx[:k] = dev(idx.astype(np.uint32).view(np.int32))
        m.val[:k] = dev(val)
    return m, {"idx": idx, "val": val.astype(np.float64)}


@pytest.mark.parametrize("n,ks", [(1, [1]), (4095, [100]), (4096, [4096]), (4097, [1, 4097]), (8192, [0, 3, 0]),
                                  (20_000, [20_000, 7, 6000]),          # every coordinate kept: beyond what is requested at once
                                  (70_001, [700] * 5), (70_001, [60, 9000] * 8), (12_289, [50] * 37),
                                  (20_000_003, [1500, 400_000])])       # several tiles per workgroup
@pytest.mark.parametrize("offset", [0, 1])
def test_entrywise_messages(n, ks, offset):
    rng = np.random.default_rng(n + len(ks))
    pairs = [entrywise(rng, n, k) for k in ks]
    out = torch.full((n + 4,), 9.0, device="cuda")
    binding.atomo_decode(ctx(), [m for m, _ in pairs], scale=0.5, out=out[offset:offset + n])
    got = out.cpu().numpy()
    want = np.zeros(n, dtype=np.float32)
    for _, h in pairs:                                                  # the order of the call, in float32
        want[h["idx"]] += np.float32(0.5) * h["val"].astype(np.float32)
    assert np.array_equal(got[offset:offset + n], want)
    assert (got[:offset] == 9).all() and (got[offset + n:] == 9).all()  # nothing beside the output is written
    np.testing.assert_allclose(got[offset:offset + n], oracle.decode_entrywise([h for _, h in pairs], n, scale=0.5),
                               rtol=1e-5, atol=1e-6)


@pytest.mark.parametrize("n,ks", [(4097, [3]), (9000, [9000, 10]), (70_001, [800] * 18)])
def test_lq_messages(n, ks):
    rng = np.random.default_rng(n)
    msgs, want = [], np.zeros(n, dtype=np.float32)
    for k in ks:
        idx = np.sort(rng.choice(n, size=k, replace=False)).astype(np.uint32)
        neg = rng.random(k) < 0.5
        m = binding.alloc_lq_message(n, k, "cuda")
        m.count.fill_(k)
        m.idx[:] = dev((idx | (neg.astype(np.uint32) << 31)).view(np.int32))
        norm = np.float32(rng.random() + 0.5)
        m.norm.fill_(float(norm))
        msgs.append(m)
        want[idx] += np.where(neg, -1, 1).astype(np.float32) * (np.float32(0.25) * norm)
    got = binding.atomo_decode(ctx(), msgs, scale=0.25).cpu().numpy()
    assert np.array_equal(got, want)


@pytest.mark.parametrize("n,k", [(3, 2), (5000, 300), (70_001, 70_001), (20_000_003, 400_000)])
@pytest.mark.parametrize("beside", [0, 3, 17])                          # messages in order that are decoded with it
@pytest.mark.parametrize("lq", [False, True])
def test_coordinates_that_do_not_ascend_are_reported(n, k, beside, lq):
    rng = np.random.default_rng(n + beside)

    def message(words):
        m = (binding.alloc_lq_message if lq else binding.alloc_entrywise_message)(n, words.size, "cuda")
        m.count.fill_(words.size)
        if lq:                                                          # (the sign bit is no part of the coordinate)
            words = words | ((rng.random(words.size) < 0.5).astype(np.uint32) << 31)
            m.norm.fill_(1.0)
        m.idx[:] = dev(words.astype(np.uint32).view(np.int32))
        return m

    good = np.sort(rng.choice(n, size=k, replace=False)).astype(np.uint32)
    others = [message(good[: max(1, k // 50)]) for _ in range(beside)]
    assert ctx().status()[0] == 0
    binding.atomo_decode(ctx(), others + [message(good)])
    assert ctx().status()[0] == 0
    for where in (0, (k - 1) // 2, k - 2):
        swapped = good.copy()
        swapped[[where, where + 1]] = swapped[[where + 1, where]]
        twice = good.copy()
        twice[where + 1] = twice[where]
        for bad in (swapped, twice, np.roll(good, k // 2)):
            binding.atomo_decode(ctx(), others + [message(bad)])
            assert ctx().status()[0] == binding.ATOMO_EINVAL
    assert ctx().status()[0] == 0                                       # (reported once)


@pytest.mark.parametrize("n,k", [(1, 0), (1, 1), (4096, 0), (4097, 4097), (12_293, 300), (1 << 22, 1 << 21), ((1 << 22) + 1, 65_536),
                                 ((1 << 22) + 1, 65_537), (8192 * 4096, 8192 * 64), (8192 * 4096 + 1, 8192 * 64)])
@pytest.mark.parametrize("offset", [0, 1])
@pytest.mark.parametrize("lq", [False, True])
def test_one_message_on_both_sides_of_its_own_kernel(n, k, offset, lq):
    """Values are stored over zeros that other waves have just stored: every output is compared, over what the buffer held before."""
    gen = torch.Generator(device="cuda").manual_seed(n + k)
    at = torch.unique(torch.randint(0, n, (k,), generator=gen, device="cuda")) if k < n else torch.arange(n, device="cuda")
    if k:
        at[0], at[-1] = 0, n - 1
    kept = at.numel() if n > 1 else k
    at = at[:kept]
    out = torch.full((n + 2,), 9.0, device="cuda")
    want = torch.full((n + 2,), 9.0, device="cuda")
    want[offset:offset + n] = 0.0
    if lq:
        m = binding.alloc_lq_message(n, max(k, 1), "cuda")
        neg = torch.rand(kept, generator=gen, device="cuda") < 0.5
        m.idx[:kept] = torch.where(neg, at - (1 << 31), at).to(torch.int32)
        m.norm.fill_(1.5)
        want[offset + at] = torch.where(neg, -0.75, 0.75)
    else:
        m = binding.alloc_entrywise_message(n, max(k, 1), "cuda")
        m.idx[:kept] = at.to(torch.int32)
        m.val[:kept] = torch.randn(kept, generator=gen, device="cuda")
        want[offset + at] = 0.5 * m.val[:kept]
    m.count.fill_(kept)
    binding.atomo_decode(ctx(), [m], scale=0.5, out=out[offset:offset + n])
    assert torch.equal(out, want)
    assert ctx().status()[0] == 0


@pytest.mark.parametrize("lq", [False, True])
@pytest.mark.parametrize("n", [96_000_000 - 1, 96_000_000 + 3])
@pytest.mark.parametrize("messages, offset", [(1, 0), (3, 0), (3, 1), (5, 0)])
def test_outputs_written_around_the_last_cache(n, messages, offset, lq):
    """From 96 million outputs of one to four messages on.  Against a sum of the messages in their order, in fp32 on the device: the same bits."""
    gen = torch.Generator(device="cuda")
    gen.manual_seed(messages)
    want, msgs = torch.zeros(n, device="cuda"), []
    for j in range(messages):
        idx = torch.randint(0, n, (200_000 * (j + 1),), generator=gen, device="cuda")
        idx[:3] = torch.tensor([0, n - 1, n - 4], device="cuda")
        idx = torch.unique(idx)
        val = torch.randn(idx.numel(), generator=gen, device="cuda")
        m = (binding.alloc_lq_message if lq else binding.alloc_entrywise_message)(n, idx.numel(), "cuda")
        m.count.fill_(idx.numel())
        if lq:
            m.norm.fill_(0.5 + j)
            m.idx.copy_((idx | (val < 0).long() << 31).to(torch.int32))
            val = torch.where(val < 0, -1.0, 1.0) * (m.norm * 0.5)
        else:
            m.idx.copy_(idx.to(torch.int32))
            m.val.copy_(val)
            val = val * 0.5
        want[idx] += val                                         # (every coordinate once per message)
        msgs.append(m)
    out = torch.full((n + 4,), 9.0, device="cuda")
    binding.atomo_decode(ctx(), msgs, scale=0.5, out=out[offset:offset + n])
    assert ctx().status()[0] == 0
    assert torch.equal(out[offset:offset + n], want)
    assert bool((out[:offset] == 9).all()) and bool((out[offset + n:] == 9).all())
