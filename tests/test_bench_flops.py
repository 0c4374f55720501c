"""The FLOPs that bench.py divides by its time, against the products that the library executes, counted one by one."""
import pytest

import bench


def products(w, rerun_last=False):
    """Multiply-adds of one layer's forward: the four linear products and the two of attention (the whole s x s square)."""
    T, h, hp, fp = w["s"] * w["b"], w["h"], w["h"] // w["t"], 4 * w["h"] // w["t"]
    n = T * h * 3 * hp + T * hp * h + T * h * fp + 2 * w["b"] * w["s"] ** 2 * hp
    return n + (0 if rerun_last else T * fp * h)


@pytest.mark.parametrize("name", sorted(bench.WORKLOADS))
@pytest.mark.parametrize("seg", [0, 1, 2, 3, 4])
def test_executed_flops(name, seg):
    w = bench.WORKLOADS[name]
    n = w["layers"]
    if seg > n:
        pytest.skip("more layers in a segment than in the chunk")
    want = 3 * n * products(w)                 # forward, and two products for each one in the backward
    for l in range(n if seg else 0):           # the rerun of each segment stops in front of its last layer's second MLP product
        want += products(w, rerun_last=(l + 1) % seg == 0 or l + 1 == n)
    assert bench.executed_flops(w, seg, 1) == 2 * want
    assert bench.executed_flops(w, seg, 16) == 32 * want
