"""The forward-only calls give the training forward's rows bit for bit although their GEMM launches
take other tile shapes: a training forward of 97,200 cells runs 128-row tiles, its context call the
same, and query chunks of 81, 405 and 2,835 cells run 32- and 64-row tiles; one of 55,080 cells runs
128- and 64-row tiles by the width.  The gradients at 55,000 cells, where tiles of both heights run
in one backward, agree with the float64 oracle.  The weight gradients at
E = 256 agree with the float64 oracle on both sides of the cell count from which their tiles are
256 wide, within the parity tests' bfloat16 tolerance (2e-2 of each tensor's largest value)."""

import numpy as np
import pytest

from paper_2606_03681_amd import workloads as wl

from _harness import compare_all, gpu_stack, oracle_stack, storage_of

pytestmark = pytest.mark.gpu

# block, E, heads, H
CASES = [("post", 192, 6, 768), ("post", 64, 2, 128), ("pre", 256, 4, 768), ("pre", 128, 2, 384)]


@pytest.mark.parametrize("R", [1200, 680])
@pytest.mark.parametrize("block,E,heads,H", CASES)
def test_rows_do_not_depend_on_tile_shape(monkeypatch, block, E, heads, H, R):
    import torch
    from paper_2606_03681_amd import tfm
    from paper_2606_03681_amd.stack import InferStack, Stack, to_device
    n, C = 500, 80
    cfg = dict(name="shape", dtype="bf16", B=1, R=R, n_train=n, C=C, E=E, heads=heads, H=H,
               layers=1, cells="normal", weights="xavier_bias", block=block)
    monkeypatch.setitem(wl.TEST_CONFIGS, "shape", cfg)
    w = wl.make_workload("shape", with_dY=False)

    def dims(rows):
        return tfm.make_dims(1, rows, C, E, heads, H, "bf16", block)

    full = storage_of(Stack(dims(R), w.n_train, w.cell_mask, w.params).forward(
        to_device(w.X, "bf16")), "bf16")
    cuts = [R - 41, R - 40, R - 35, R]                  # query chunks of 1, 5 and 35 rows
    inf = InferStack(dims(cuts[0]), w.n_train, w.cell_mask, w.params, max_query_rows=40)
    got = [storage_of(inf.context(to_device(np.ascontiguousarray(w.X[:, :cuts[0]]), "bf16")),
                      "bf16")]
    for a, b in zip(cuts, cuts[1:]):
        got.append(storage_of(inf.query(to_device(np.ascontiguousarray(w.X[:, a:b]), "bf16")),
                              "bf16"))
    torch.cuda.synchronize()
    assert np.array_equal(np.concatenate(got, axis=1), full)


# 49,300, 55,020 and 65,520 cells: the two ends of the range in which single-column launches take
# 128 rows below GEMM_FILL tiles, and its middle
@pytest.mark.parametrize("block,E,heads,H,B,R,C", [("post", 192, 12, 384, 4, 725, 16),
                                                   ("pre", 192, 6, 192, 4, 655, 20),
                                                   ("pre", 256, 16, 256, 6, 546, 19)])
def test_gradients_where_one_round_of_tall_tiles_suffices(monkeypatch, block, E, heads, H, B, R, C):
    cfg = dict(name="once", dtype="bf16", B=B, R=R, n_train=(1, R), C=C, E=E, heads=heads, H=H,
               layers=1, cells="normal", weights="xavier_bias", block=block)
    monkeypatch.setitem(wl.TEST_CONFIGS, "once", cfg)
    w = wl.make_workload("once")
    compare_all(w, gpu_stack(w), oracle_stack(w))


# block, B, R, n_train, C, active, H: 20,000 cells (one column spans less than a slice of the
# contraction), 19,980 and ragged tables of more than 21,000
WIDE = [("post", 100, 20, (1, 20), 9, None, 256), ("post", 2, 999, 700, 9, None, 512),
        ("pre", 2, 703, (1, 703), 21, (16, 21), 768)]


@pytest.mark.parametrize("block,B,R,n,C,active,H", WIDE)
def test_weight_gradients_at_width_256(monkeypatch, block, B, R, n, C, active, H):
    cfg = dict(name="wide", dtype="bf16", B=B, R=R, n_train=n, C=C, E=256, heads=8, H=H, layers=1,
               cells="normal", weights="xavier_bias", block=block)
    if active:
        cfg.update(active=active, mask="random")
    monkeypatch.setitem(wl.TEST_CONFIGS, "wide", cfg)
    w = wl.make_workload("wide")
    compare_all(w, gpu_stack(w), oracle_stack(w))
