"""GPU checks of the chunked form's blocks: trees of one slot up to one past a
block's edge, last blocks cut off by the tree and by T, one, two and three
earlier blocks with ancestors (the cascade takes two at a time) and earlier
blocks without any, more value heads per key head than a workgroup has waves,
head sizes with idle waves; against the CPU oracle."""
import numpy as np
import pytest

from paper_2607_06763_amd import workloads as W

pytestmark = pytest.mark.gpu

# Operands are bf16 hi + lo, 2^-16 per product; a result gathers a few products
# in a row (Gram block, update, S0 product), each times at most a few such sums.
O_TOL = 16 * 2.0 ** -16


@pytest.fixture(scope="module")
def G():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2607_06763_amd import gdn_tree as G
    G.lib()
    return G


def _tree(T, n, stem, skip):
    """A chain of `stem` nodes, then `skip` leaves of its first node, then a
    chain below its last one: blocks of leaves hold no ancestors."""
    par = np.full(T, W.PAD, np.int32)
    for i in range(n):
        par[i] = W.ROOT if i == 0 else i - 1 if i < stem else 0 if i < stem + skip else i - 1 if i > stem + skip else stem - 1
    return par


@pytest.mark.parametrize("T,n,stem,skip,Hk,Hv,dk,dv,dtype", [
    (1, 1, 1, 0, 1, 1, 16, 16, "f32"),
    (31, 31, 31, 0, 1, 2, 32, 16, "bf16"),
    (32, 32, 32, 0, 3, 3, 16, 128, "f32"),
    (33, 33, 33, 0, 1, 3, 128, 32, "bf16"),
    (64, 33, 33, 0, 2, 2, 64, 64, "f32"),
    (97, 96, 96, 0, 1, 10, 32, 32, "bf16"),     # three earlier blocks; 10 value heads of a key head
    (100, 70, 70, 0, 3, 6, 128, 128, "f32"),    # blocks past the tree, 9 units on 8 XCDs
    (160, 150, 20, 80, 1, 2, 64, 128, "bf16"),  # ancestors in the first block and the last two only
    (512, 511, 200, 150, 1, 1, 128, 64, "bf16"),
])
def test_blocks(G, orc, T, n, stem, skip, Hk, Hv, dk, dv, dtype):
    import torch
    bad = np.full(T, W.PAD, np.int32)
    bad[0] = 0  # its own parent
    par = np.stack([_tree(T, n, stem, skip), bad, W.random_tree(np.random.default_rng(T + n), T, n)])
    w = W.make_random(9300 + T + n, 3, T, Hk, Hv, dk, dv, dtype, parent=par)
    print(f"[gpu] chunked blocks T={T} n={n} stem={stem} skip={skip} {Hk}/{Hv} heads {dk}x{dv}", flush=True)
    dt = G.DeviceTree(w)
    dt.prepare()
    out = torch.full_like(dt.out, float("nan"))
    dt.verify(out=out, chunked=True)
    torch.cuda.synchronize()
    ref, got = orc.verify(w), out.cpu().numpy()
    err = np.max(np.abs(got - ref)) / np.max(np.abs(ref))
    print(f"[gpu]   err {err:.3e}", flush=True)
    assert err <= O_TOL
    assert (got[1] == 0).all() and (got[0, n:] == 0).all()
