"""GPU parity of the float32-arithmetic path (float32 storage, and bfloat16 shapes outside the
bf16 matrix-core envelope) at the edges of its tiles: widths that are not multiples of the 64-wide
product tiles, fewer cells than one tile or one chunk of the weight gradients, more cells than
the chip has chunks for, train prefixes of 1 and R, inactive columns, every head width.  Against
the float64 oracle with the tolerances of the parity tests (float32 arithmetic: 1e-4 of each
tensor's largest value; bfloat16 storage: 2e-2)."""

import pytest

from paper_2606_03681_amd import workloads as wl

from _harness import compare_all, gpu_stack, oracle_stack

pytestmark = pytest.mark.gpu

# dtype, B, R, n_train, C, active, E, heads, H
CASES = [
    ("f32", 1, 1, 1, 0, None, 32, 2, 32),            # one cell
    ("f32", 1, 5, 3, 1, None, 32, 1, 32),            # fewer cells than any tile
    ("f32", 3, 33, (1, 33), 4, (0, 4), 96, 3, 160),  # widths between the 64-wide tiles
    ("f32", 2, 65, (1, 65), 6, (0, 6), 160, 10, 96),  # head width 16, rows one past a tile
    ("f32", 2, 40, 17, 3, None, 224, 7, 352),
    ("f32", 1, 130, 129, 2, None, 256, 4, 1024),     # the widest block, head width 64
    ("f32", 3, 900, (1, 900), 15, (3, 15), 32, 1, 64),  # several cells per chunk and tile
    ("f32", 4, 20, (1, 20), 150, (130, 150), 32, 2, 32),  # rows of more than 128 cells
    ("f32", 110, 3, (1, 3), 2, (0, 2), 32, 2, 32),   # a plan too long for kernel arguments
    ("bf16", 3, 70, (1, 70), 5, (0, 5), 96, 3, 96),  # bfloat16 widths without a bf16 path
    ("bf16", 2, 31, 30, 3, None, 192, 6, 96),        # H not a multiple of E
]


@pytest.mark.parametrize("dtype,B,R,n,C,active,E,heads,H", CASES)
def test_f32_path_edges(monkeypatch, dtype, B, R, n, C, active, E, heads, H):
    cfg = dict(name="edge", dtype=dtype, B=B, R=R, n_train=n, C=C, E=E, heads=heads, H=H,
               layers=1, cells="normal", weights="xavier_bias")
    if active:
        cfg.update(active=active, mask="random")
    monkeypatch.setitem(wl.TEST_CONFIGS, "edge", cfg)
    w = wl.make_workload("edge")
    compare_all(w, gpu_stack(w), oracle_stack(w))


@pytest.mark.parametrize("name", ["d64-f32", "d64-bf16", "prenorm-small-bf16"])
@pytest.mark.parametrize("shared", ["X", "dY"])
def test_dX_may_share_memory_with_an_input(name, shared):
    """The backward of one layer with dX written over X (post-norm) or dY gives the gradients of
    the call with a buffer of its own, bit for bit."""
    import torch
    from paper_2606_03681_amd import tfm
    from paper_2606_03681_amd.stack import Stack, to_device
    w = wl.make_workload(name)
    dims = tfm.make_dims(dtype=w.dtype, block=w.block,
                         **{k: v for k, v in w.dims.items() if k != "dtype"})
    got = []
    for inplace in (False, True):
        st = Stack(dims, w.n_train, w.cell_mask, w.params[:1])
        X, dY = to_device(w.X, w.dtype), to_device(w.dY, w.dtype)
        st.forward(X)
        out = st.dxs[0] if not inplace else (X if shared == "X" else dY)
        tfm.layer_bwd(st.layer_dims[0], st.n_train, st.cell_mask, X, st.params[0], st.saved[0],
                      dY, out, st.grads[0], False, st.workspace)
        torch.cuda.synchronize()
        got.append((out.clone(), st.grads[0].clone()))
    for a, b in zip(*got):
        assert torch.equal(a, b)


def _overflow_inputs(dtype, axis, n, C, E, heads):
    """One table whose attention along `axis` scores -infinity in float32 (a product of 1e40) against
    the first half of the keys and 0 against the others: feature 0 of a cell is -1 or 0 (over the
    others, +-1 in turn), Q holds 1e20 and K 1e20 times that feature of its norm-1 input."""
    import numpy as np
    rng = np.random.default_rng(3)
    R = n + 3
    prm = wl._draw_params(rng, E, 64, "xavier_bias")
    at, views = 0, {}
    for name, shape, _ in wl.param_layout(E, 64):
        k = int(np.prod(shape))
        views[name] = prm[at:at + k].reshape(shape)
        at += k
    ax = "f" if axis == "feature" else "i"
    W, b = views["Wqkv_" + ax], views["bqkv_" + ax]
    W[:2 * E] = 0
    b[:2 * E] = 0
    d = E // heads
    for h in range(heads):
        b[h * d] = 1e20
        W[E + h * d, 0] = 1e20
    if axis == "item":  # the item axis reads LN1(X + 0): no output of the feature axis
        views["Wo_f"][:] = 0
        views["bo_f"][:] = 0
        views["g1"][0], views["be1"][0] = 1, 0
    X = np.ones((1, R, C + 1, E))
    X[..., 1::2] = -1
    X[..., 0], X[..., -1] = 0, 0
    low = (np.arange(R) < n // 2)[:, None] if axis == "item" else (np.arange(C + 1) < C // 2)[None]
    X[0, ..., 0] = np.where(low, -1, 0)
    X[0, ..., -1] = np.where(low, 1, 0)
    return wl.to_storage(X, dtype), prm, np.array([n], np.int32), R


@pytest.mark.parametrize("dtype,axis,n,C,heads", [("f32", "item", 80, 2, 6), ("f32", "item", 70, 1, 3),
                                                  ("f32", "feature", 5, 70, 3),
                                                  ("bf16", "feature", 5, 90, 6)])
def test_first_key_tiles_of_overflowing_scores(dtype, axis, n, C, heads):
    """Keys whose scores are -infinity have probability 0, also where every key of the first tiles
    is one: the forward equals the oracle's, in which they are -1e40."""
    import numpy as np
    import oracle
    import torch
    from _harness import TOL, nerr
    from paper_2606_03681_amd import tfm
    from paper_2606_03681_amd.stack import Stack, to_device, to_host
    E = 96
    X, prm, nt, R = _overflow_inputs(dtype, axis, n, C, E, heads)
    mask = np.ones((1, C + 1), np.uint8)
    P = oracle.unpack_params(prm.astype(np.float64), E, 64)
    ref, _ = oracle.stack_forward(wl.storage_to_f64(X, dtype), [P], nt, mask, heads)
    Y = Stack(tfm.make_dims(1, R, C, E, heads, 64, dtype), nt, mask, [prm]).forward(
        to_device(X, dtype))
    got = to_host(Y, dtype)
    torch.cuda.synchronize()
    assert nerr(got, ref) <= TOL[dtype]


@pytest.mark.parametrize("axis", ["item", "feature"])
@pytest.mark.parametrize("E,heads", [(32, 2), (96, 3), (128, 2)])
def test_probabilities_of_large_scores(axis, E, heads):
    """A key that dominates has probability 1 in the backward too, whatever its score: with one key
    and scores of some 1e6 the value gradients are those of the oracle.  (A probability from a
    rounded log-sum-exp is off by the score's rounding, 0.1 there.)"""
    import numpy as np
    import torch
    from _harness import TOL, nerr
    import oracle
    from paper_2606_03681_amd import tfm
    from paper_2606_03681_amd.stack import Stack, to_device
    rng = np.random.default_rng(11)
    B, R, H, n = 3, 50, 64, (1 if axis == "item" else 20)
    C = 0 if axis == "feature" else 2
    prm = wl._draw_params(rng, E, H, "xavier_bias")
    at = 0
    for name, shape, _ in wl.param_layout(E, H):
        k = int(np.prod(shape))
        if name == ("bqkv_i" if axis == "item" else "bqkv_f"):
            prm[at:at + 2 * E] *= 5000
        at += k
    X = rng.normal(size=(B, R, C + 1, E)).astype(np.float32)
    dY = rng.normal(size=X.shape).astype(np.float32)
    nt, mask = np.full(B, n, np.int32), np.ones((B, C + 1), np.uint8)
    st = Stack(tfm.make_dims(B, R, C, E, heads, H, "f32"), nt, mask, [prm])
    st.forward(to_device(X, "f32"))
    st.backward(to_device(dY, "f32"))
    torch.cuda.synchronize()
    got = oracle.unpack_params(st.grads[0].double().cpu().numpy(), E, H)
    Y, caches = oracle.stack_forward(X.astype(np.float64), [oracle.unpack_params(
        prm.astype(np.float64), E, H)], nt, mask, heads)
    _, (want,) = oracle.stack_backward(dY.astype(np.float64), caches)
    ax = "i" if axis == "item" else "f"
    for name in ("Wqkv_" + ax, "bqkv_" + ax):
        assert nerr(got[name][2 * E:], want[name][2 * E:]) <= TOL["f32"], name
