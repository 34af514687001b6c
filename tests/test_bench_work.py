"""CPU checks of the work model of bench.py: every kernel class that an SVD step can launch has a price, and a layer is
priced by the route that it reports."""
import numpy as np
import pytest

import bench
from paper_1806_04090_amd import binding, inputs


def work(shapes, sweeps, refreshes, kept=None):
    n = sum(m * k for m, k in shapes)
    return bench.executed_work(shapes, sweeps, refreshes, 0, 0, 0, n, kept or [3] * len(shapes))


def test_every_kernel_class_of_an_svd_step_has_a_price():
    shapes = list(inputs.RESNET18_SHAPES)
    priced = work(shapes, [1] * len(shapes), [2] * len(shapes))
    for name in binding.Context.KERNEL_CLASSES:
        if name.startswith("svd_") or name == "decode_svd":
            bound, amount, peak, unit = priced[name]
            assert amount >= 0 and peak > 0 and unit in ("TFLOP/s", "GB/s"), name


@pytest.mark.parametrize("shape", [(64, 576), (512, 4608), (640, 700)])
def test_a_layer_is_priced_by_the_route_it_reports(shape):
    m, n = shape
    direct, iterated = work([shape], [1], [2]), work([shape], [7], [3])
    assert direct["svd_refresh"][1] == 0 and direct["svd_update"][1] == 0 and iterated["svd_direct"][1] == 0
    np.testing.assert_allclose(direct["svd_direct_gram"][1], n * m * (m + 64.0))
    np.testing.assert_allclose(direct["svd_direct"][1], n * m * (m + 64.0) + 2.0 * m ** 3 + 3 * 2.0 * m * (m + n))
    assert bench.dense_equivalent_flops([shape], [1], [2]) == 0 < bench.dense_equivalent_flops([shape], [7], [3])
    flops, peak = bench.matrix_core_work(direct, 0.0)
    assert flops == direct["svd_direct_gram"][1] and peak == pytest.approx(bench.PEAK_FP64_TFLOPS)
    flops, peak = bench.matrix_core_work(iterated, 0.0)
    assert flops > 0 and peak == pytest.approx(bench.PEAK_FP32_MFMA_TFLOPS)


def test_a_long_gradient_is_priced_as_one_read():
    # the encoder's own limit, as the source has it
    import os
    import re
    source = open(os.path.join(os.path.dirname(bench.__file__), "paper_1806_04090_amd", "csrc", "entrywise.hip")).read()
    assert bench.SAMPLED_FROM == 1 << int(re.search(r"constexpr long long LONG_FROM = 1ll << (\d+);", source)[1])
    assert bench.entrywise_bytes(2 ** 25 - 1, 0) == 12 * (2 ** 25 - 1) and bench.entrywise_bytes(2 ** 25, 0) == 8 * 2 ** 25
    assert bench.entrywise_bytes(2 ** 30, 10) == 8 * 2 ** 30 + 200
