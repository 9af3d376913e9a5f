"""Batches of many tables of few rows or cells, whose attention takes 2^32 threads and more: one launch
of that size starts only what is left modulo 2^32, so the kernels go in pieces.  Every dataset's rows
are bit for bit those of a call on that dataset alone, forward and backward."""

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

# what needs the pieces, its threads (a lower bound, from the arguments below), dtype, block, B, R,
# n_train, C, E, heads, H, the datasets to run again alone
MANY = [
    # float32 arithmetic: 256 threads for 64 rows of a (column, head) problem; a wave for 16 cells
    # of a (row, head) pair
    ("item", lambda B, R, S, h: B * S * h * 256, "f32", "post", 8193, 2, (1, 2), 255, 128, 8, 32,
     (0, 4100, 8192)),
    ("feature", lambda B, R, S, h: B * R * h * 64, "bf16", "post", 3, 1597831, (1, 9), 0, 224, 14,
     32, (0, 2)),
    # bfloat16 matrix-core kernels: 256 threads a problem forward, 512 in the one-kernel backward;
    # 256 in each kernel of the two-kernel backward (head width 64); a wave a (row, head) pair
    ("item, one kernel", lambda B, R, S, h: B * S * h * 256, "bf16", "post", 16385, 2, (1, 2), 127,
     128, 8, 128, (0, 8200, 16384)),
    ("item, two kernels", lambda B, R, S, h: B * S * h * 256, "bf16", "pre", 32769, 1, (1, 1), 127,
     256, 4, 256, (0, 20000, 32768)),
    ("feature", lambda B, R, S, h: B * R * h * 64, "bf16", "post", 3, 5592411, (1, 9), 0, 64, 4, 64,
     (0, 2)),
]


@pytest.mark.parametrize("what,threads,dtype,block,B,R,n,C,E,heads,H,picks", MANY)
def test_many_tables(what, threads, dtype, block, B, R, n, C, E, heads, H, picks):
    import torch
    from paper_2606_03681_amd import tfm
    from paper_2606_03681_amd.stack import Stack
    assert threads(B, R, C + 1, heads) >= 1 << 32
    gen = torch.Generator(device="cuda").manual_seed(17)
    elt = torch.float32 if dtype == "f32" else torch.bfloat16
    nt = np.random.default_rng(17).integers(n[0], n[1] + 1, B).astype(np.int32)
    mask = np.ones((B, C + 1), np.uint8)

    def dims(b):
        return tfm.make_dims(b, R, C, E, heads, H, dtype, block)

    def layer(b, X, dY, prm):
        st = Stack(dims(len(nt[b])), nt[b], mask[b], [prm])
        return st.forward(X[b]), st.backward(dY[b])

    X = torch.empty((B, R, C + 1, E), device="cuda", dtype=elt).normal_(generator=gen)
    dY = torch.empty_like(X).normal_(generator=gen)
    prm = torch.randn(tfm.param_count(dims(B)), generator=gen, device="cuda") * 0.1
    Y, dX = layer(slice(None), X, dY, prm)
    torch.cuda.synchronize()
    for b in picks:
        y, dx = layer(slice(b, b + 1), X, dY, prm)
        assert bool(torch.isfinite(y).all()) and bool(torch.isfinite(dx).all())
        assert torch.equal(y[0], Y[b]) and torch.equal(dx[0], dX[b]), b
    del X, dY, Y, dX
    torch.cuda.empty_cache()


def test_thinking_rows_of_many_tables():
    """More than 2^32 elements of thinking rows, one thread each."""
    import torch
    from paper_2606_03681_amd import tfm
    B, R, C, E, T = 131073, 1, 127, 256, 1
    dims = tfm.make_dims(B, R, C, E, 4, 256, "bf16", "pre")
    assert B * T * (C + 1) * E > 1 << 32
    nt = np.ones(B, np.int32)
    mask = np.ones((B, C + 1), np.uint8)
    mask[B - 1, 0] = 0
    table = torch.randn((T, E), device="cuda")
    X = torch.full((B, R, C + 1, E), 3.0, device="cuda", dtype=torch.bfloat16)
    ws = torch.empty(tfm.infer_workspace_bytes(tfm.make_dims(B, R, C, 64, 4, 64, "bf16")),
                     dtype=torch.uint8, device="cuda")
    tfm.thinking_rows_fwd(dims, nt, mask, T, table, X, ws)
    want = table.to(torch.bfloat16)[0]
    assert bool((X[:-1] == want).all())
    assert bool((X[-1, 0, 1:] == want).all()) and bool((X[-1, 0, 0] == 0).all())
    del X, ws
    torch.cuda.empty_cache()
