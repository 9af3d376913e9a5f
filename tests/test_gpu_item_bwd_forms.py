"""The item-attention backward in each of its forms: one kernel with 256, 512 or 768 keys, two kernels,
and both in one call, at the head widths that have them.  Each case states the form that the call's
column count and prefixes lead to, checked from the steps that ran; results against the float64
oracle within the parity tests' bfloat16 tolerance (2e-2 of each tensor's largest value)."""

import numpy as np
import pytest

from paper_2606_03681_amd import workloads as wl

from _harness import compare_all, gpu_stack, oracle_stack

pytestmark = pytest.mark.gpu

ONE, TWO, BOTH = "one", "two", "both"
# E, heads, B, R, n_train of the tables between the first (1) and the last (R), C, form, longest
# prefix in the one-kernel form
CASES = [
    (64, 4, 6, 256, (100, 256), 9, ONE, 256),     # d = 16: 2, 4 and 6 key blocks a wave
    (64, 4, 9, 512, (257, 512), 9, ONE, 512),
    (64, 4, 9, 768, (513, 768), 9, ONE, 768),
    (64, 4, 12, 900, (200, 900), 9, BOTH, 768),
    (64, 4, 3, 700, (300, 700), 3, TWO, 0),       # too few columns to fill it
    (192, 6, 7, 257, (200, 257), 9, ONE, 257),    # d = 32
    (64, 2, 12, 768, (513, 768), 11, ONE, 768),
    (64, 2, 3, 700, (300, 700), 3, TWO, 0),
    (128, 2, 5, 300, (100, 300), 9, TWO, 0),      # d = 64 has no one-kernel form
]


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.fail("no GPU visible")
    from paper_2606_03681_amd import tfm
    tfm.lib()


def _ran(prof):
    one = any(k.startswith("item_attn_bwd/") for k in prof)
    two = any(k.startswith("item_attn_dq/") for k in prof)
    assert two == any(k.startswith("item_attn_dkdv/") for k in prof)
    return BOTH if one and two else ONE if one else TWO


def _run(w):
    from paper_2606_03681_amd import tfm
    tfm.prof_enable(True)
    try:
        gpu = gpu_stack(w)
        form = _ran(tfm.prof_collect())
    finally:
        tfm.prof_enable(False)
    return gpu, form


@pytest.mark.parametrize("E,heads,B,R,n,C,form,longest", CASES)
def test_form(monkeypatch, E, heads, B, R, n, C, form, longest):
    cfg = dict(name="form", dtype="bf16", B=B, R=R, n_train=n, C=C, active=(C // 2, C),
               mask="random", E=E, heads=heads, H=2 * E, layers=1, cells="normal",
               weights="xavier_bias")
    monkeypatch.setitem(wl.TEST_CONFIGS, "form", cfg)
    w = wl.make_workload("form")
    gpu, ran = _run(w)
    assert ran == form
    if longest:  # the tables reach into the key range that the case stands for
        top = max(x for x in w.n_train if x <= 768)
        assert longest - 256 < top <= longest
    compare_all(w, gpu, oracle_stack(w))


def test_mixed_prefix_workload_runs_both_forms():
    """The parity and accumulation tests take this workload for the split of one call's columns."""
    w = wl.make_workload("mixed-prefix-bf16")
    assert _run(w)[1] == BOTH
    short = np.repeat(w.n_train, w.cell_mask.sum(1, dtype=np.int64)) <= 768
    assert short.sum() == 30 and len(short) == 60
