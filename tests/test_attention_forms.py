"""Every form of the bf16 attention kernels that a call can take is run by a GPU test against the oracle.

The forms follow from the sizes by host-side rules (ptdp_attn_form); this test runs them over the whole range of sizes and
over the parameter lists of the GPU tests.  Kinds: the causal mask; no mask; a general mask whose rows are a multiple of four
bytes; one whose rows are not."""
import ctypes as C

import pytest

import test_gpu_gemm_attn as causal_tests
import test_gpu_masked_attention as masked_tests
from paper_2104_04473_amd import binding as B

HEAD_SIZES = (32, 64, 96, 128, 160)
KERNELS = ("forward", "dQ", "dK/dV")


def form(kernel, kind, s, b, heads, dh):
    v = [C.c_int() for _ in range(4)]
    call = (int(kind == "causal"), int(kind.startswith("mask")), s, b, heads, dh)
    B.check(B.ptdp_attn_form(kernel, *call, *[C.byref(x) for x in v]), "form")
    if kernel > 0:   # backward: also whether dQ and dK/dV share a launch, and whether dK and dV have waves of their own
        launch = [C.c_int(), C.c_int()]
        B.check(B.ptdp_attn_bwd_launch(*call, *[C.byref(x) for x in launch]), "launch")
        v += launch
    return tuple(x.value for x in v)


def params(fn):
    return [p for mark in fn.pytestmark if mark.name == "parametrize" for p in mark.args[1]]


def forms_run():
    cases = [("causal", c[1:]) for c in causal_tests.ATTN_CASES if c[0] == B.BF16]
    cases += [("causal", c) for c in params(causal_tests.test_attention_forms)]
    masked = [(c[1:5], c[5]) for c in masked_tests.CASES if c[0] == B.BF16]
    masked += [(c, True) for c in params(masked_tests.test_masked_attention_forms)]
    masked += [(c, False) for c in params(masked_tests.test_unmasked_attention_forms)]
    cases += [("none" if not m else "mask bytes" if c[0] % 4 else "mask words", c) for c, m in masked]
    return {(kernel, kind, c[3], form(kernel, kind, *c)) for kind, c in cases for kernel in range(3)}


@pytest.mark.parametrize("kind", ["causal", "none", "mask words", "mask bytes"])
@pytest.mark.parametrize("dh", HEAD_SIZES)
def test_every_form_is_run(kind, dh):
    have = forms_run()
    pairs = [1, 2, 3, 5, 8, 13, 16, 24, 40, 64, 100, 128, 160, 200, 256, 300, 400, 512, 600, 800, 1000, 1300, 2000, 4100, 10000]
    want = {}
    for s in list(range(1, 200, 3)) + [4 * k for k in range(1, 50)] + [257, 260, 321, 324, 384, 385, 388, 449, 452, 513, 516, 777, 1024, 1027, 2048,
                                                                        4096, 4099, 16384]:
        if kind.startswith("mask") and (s % 4 == 0) != (kind == "mask words"):
            continue
        for p in pairs:
            for kernel in range(3):
                want.setdefault((kernel, kind, dh, form(kernel, kind, s, 1, p, dh)), (s, p))
    missing = sorted((KERNELS[k[0]], k[3], example) for k, example in want.items() if k not in have)
    assert not missing, "no GPU test runs (kernel, (rows, groups, tile, wide (, together, split)), an example of s and heads): %s" % missing


@pytest.mark.parametrize("dh", [32, 64, 96, 128])
@pytest.mark.parametrize("kind", ["causal", "none", "mask words", "mask bytes"])
def test_short_sequences_of_many_heads_take_small_workgroups(kind, dh):
    """Up to 64 rows per head, and 129 to 160: no workgroup of 128 rows that is half empty or more."""
    for s in (33, 36, 63, 64, 129, 132, 157, 160):
        if kind.startswith("mask") and (s % 4 == 0) != (kind == "mask words"):
            continue
        for heads in (1024, 4096):
            for kernel in range(3):
                rows, groups = form(kernel, kind, s, 1, heads, dh)[:2]
                assert rows == 64 and (groups == 1 or kind == "mask bytes"), (s, heads, KERNELS[kernel])
