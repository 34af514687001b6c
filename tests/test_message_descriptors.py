"""CPU checks of the C descriptors of messages: they follow the message's fields, and a message that has been used can be
copied and pickled."""
import copy
import pickle

import pytest
import torch

from paper_1806_04090_amd import binding

MAKE = {
    "svd": lambda: binding.alloc_svd_message(6, 9, 4, "cpu"),
    "folded": lambda: binding.alloc_svd_message(6, 9, 4, "cpu", folded=True),
    "entrywise": lambda: binding.alloc_entrywise_message(100, 8, "cpu"),
    "lq": lambda: binding.alloc_lq_message(100, 8, "cpu"),
}
BUFFERS = {"svd": ("count", "idx", "w", "U", "V"), "folded": ("count", "idx", "U", "V"), "entrywise": ("count", "idx", "val"),
           "lq": ("count", "idx", "norm")}


def use(msg):
    """What a call hands down."""
    return binding._packed([msg]) if isinstance(msg, binding.SvdMessage) else bytes(msg.c_struct())


@pytest.mark.parametrize("kind", MAKE)
def test_an_assigned_buffer_is_the_one_that_is_used(kind):
    msg = MAKE[kind]()
    use(msg)
    for name in BUFFERS[kind]:
        other = torch.zeros_like(getattr(msg, name))
        setattr(msg, name, other)
        use(msg)
        assert getattr(msg.c_struct(), name) == other.data_ptr()
        assert use(msg) == bytes(msg.c_struct())
    msg.capacity -= 1
    assert use(msg) == bytes(msg.c_struct()) and msg.c_struct().capacity == msg.capacity
    if kind == "svd":
        msg.w = None
        assert use(msg) == bytes(msg.c_struct()) and msg.c_struct().w is None


@pytest.mark.parametrize("kind", MAKE)
@pytest.mark.parametrize("how", [copy.deepcopy, lambda m: pickle.loads(pickle.dumps(m))])
def test_a_used_message_is_copied_with_buffers_of_its_own(kind, how):
    msg = MAKE[kind]()
    use(msg)
    twin = how(msg)
    assert use(twin) == bytes(twin.c_struct()) != use(msg)
    for name in BUFFERS[kind]:
        assert torch.equal(getattr(twin, name), getattr(msg, name))
        assert getattr(twin.c_struct(), name) == getattr(twin, name).data_ptr() != getattr(msg, name).data_ptr()
    shallow = copy.copy(msg)
    use(shallow)
    shallow.idx = torch.zeros_like(msg.idx)
    assert use(shallow) == bytes(shallow.c_struct()) != use(msg) == bytes(msg.c_struct())
