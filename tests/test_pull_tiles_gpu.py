"""GPU checks of the tiled pull-back (trees above 128 slots): tiles of 16 nodes
in depth-first order, whose first node has just below, at and just above 16
and 32 ancestors, and last tiles of 1, 15 and 16 nodes; against the CPU oracle
with the bar of the other verify tests.  Values and keys that are not finite
reach the nodes below them and no others."""
import numpy as np
import pytest

from paper_2607_06763_amd import workloads as W

pytestmark = pytest.mark.gpu

O_TOL = 2e-3  # fp16 features and state plane, 11 significant bits (as in the other tests above 128 slots)


@pytest.fixture(scope="module")
def G():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2607_06763_amd import gdn_tree as G
    G.lib()
    return G


def _broom(T, n, depth):
    """A chain of `depth` nodes, the rest as leaves of its last node; slots
    reversed so that the depth-first order is not the slot order."""
    par = np.full(T, W.PAD, np.int32)
    for i in range(n):
        p = i - 1 if i <= depth else depth - 1
        par[n - 1 - i] = W.ROOT if i == 0 else n - 1 - p
    return par


@pytest.mark.parametrize("T,n,depth", [
    (129, 129, 15), (129, 129, 16), (145, 145, 17), (160, 159, 31), (160, 144, 32), (161, 161, 33),
    (200, 1, 1), (192, 177, 100), (512, 511, 16), (512, 497, 300), (130, 130, 1),
])
def test_tile_edges(G, orc, T, n, depth):
    import torch
    par = np.stack([_broom(T, n, depth), W.random_tree(np.random.default_rng(T + n), T, n)])
    w = W.make_random(9100 + T + depth, 2, T, 1, 2, 32, 64, "bf16", parent=par)
    print(f"[gpu] tiles T={T} n={n} depth={depth}", flush=True)
    dt = G.DeviceTree(w)
    dt.prepare()
    dt.verify()
    torch.cuda.synchronize()
    ref = orc.verify(w)
    err = np.max(np.abs(dt.out.cpu().numpy() - ref)) / np.max(np.abs(ref))
    print(f"[gpu]   err {err:.3e}", flush=True)
    assert err <= O_TOL


@pytest.mark.parametrize("what,value", [("v", float("inf")), ("v", float("nan")), ("k", float("nan")), ("k", float("-inf"))])
def test_not_finite_reaches_only_descendants(G, orc, what, value):
    import torch
    T = 200
    w = W.make_random(9200, 2, T, 1, 2, 32, 32, "f32", shuffle=True)
    ref = orc.prepare(w.parent)
    b, j = 1, int(np.nonzero(w.parent[1] >= 0)[0][7])
    print(f"[gpu] {what} = {value} at one node", flush=True)
    dt = G.DeviceTree(w)
    dt.prepare()
    dt.verify()
    torch.cuda.synchronize()
    clean = dt.out.clone().cpu().numpy()
    x = getattr(dt, what).clone()
    x[b, j, 0, 3] = value
    setattr(dt, what, x)
    dt.verify()
    torch.cuda.synchronize()
    got = dt.out.cpu().numpy()
    desc = np.array([i == j or (int(ref["anc"][b, i, j // 64]) >> (j % 64)) & 1 for i in range(T)], bool)
    heads = [0] if what == "v" else [0, 1]  # one value head, or both of the key head
    keep = np.ones(got.shape[:3], bool)
    for h in heads:
        assert not np.isfinite(got[b, j, h]).all()
        keep[b, desc, h] = False
    np.testing.assert_array_equal(got[keep].view(np.int32), clean[keep].view(np.int32))


def _stem_and_branch(T, anc, branch=2):
    """Root and a stem, `anc` nodes in all, leaves of its last one, and last in
    depth-first order a branch of `branch` nodes below the root: the leaves'
    tiles walk a path whose last chunk has absent rows unless 16 divides anc."""
    par = np.full(T, W.PAD, np.int32)
    for i in range(T):
        par[i] = W.ROOT if i == 0 else i - 1 if i < anc else anc - 1
    for j in range(branch):
        par[T - branch + j] = 0 if j == 0 else T - branch + j - 1
    return par


@pytest.mark.parametrize("anc", [1, 5, 15, 16, 17, 31, 40, 100])
@pytest.mark.parametrize("back,value", [(0, float("inf")), (0, float("nan")), (1, float("-inf")), (1, float("nan"))])
def test_not_finite_value_at_the_last_node(G, anc, back, value):
    """A value that is not finite at the last node in depth-first order, or at
    its parent: absent rows of a path chunk load that node's row."""
    import torch
    T = 150
    w = W.make_random(9400 + anc, 1, T, 1, 2, 32, 64, "f32", parent=_stem_and_branch(T, anc)[None])
    j = T - 1 - back
    print(f"[gpu] v = {value} at slot {j}, {anc} ancestors of the other leaves", flush=True)
    dt = G.DeviceTree(w)
    dt.prepare()
    dt.verify()
    torch.cuda.synchronize()
    clean = dt.out.clone().cpu().numpy()
    assert np.isfinite(clean).all()
    dt.v[0, j, 1, 3] = value
    dt.verify()
    torch.cuda.synchronize()
    got = dt.out.cpu().numpy()
    assert not np.isfinite(got[0, j:, 1, 3]).any()
    keep = np.ones(got.shape, bool)
    keep[0, j:, 1] = False
    np.testing.assert_array_equal(got[keep].view(np.int32), clean[keep].view(np.int32))


@pytest.mark.parametrize("value", [float("inf"), float("nan")])
def test_not_finite_value_keeps_other_channels(G, value):
    """A v~ row with one channel that is not finite: the other channels of the
    nodes below it come from the value terms of all their path rows."""
    import torch
    T = 200
    w = W.make_random(9500, 2, T, 1, 2, 32, 32, "f32", shuffle=True)
    w.S0 = np.zeros_like(w.S0)
    print(f"[gpu] v = {value} in one channel of every fifth slot", flush=True)
    dt = G.DeviceTree(w)
    dt.prepare()
    dt.verify()
    torch.cuda.synchronize()
    clean = dt.out.clone().cpu().numpy()
    dt.v[:, ::5, :, 3] = value
    dt.verify()
    torch.cuda.synchronize()
    got = dt.out.cpu().numpy()
    assert not np.isfinite(got[..., 3]).all()
    other = np.arange(32) != 3
    # the scale of such a row may be another power of two: fp16 values below
    # 2^-14 of its largest round differently, by 2^-25 of it
    err = np.max(np.abs(got[..., other] - clean[..., other])) / np.max(np.abs(clean))
    assert err <= 1e-5


@pytest.mark.parametrize("ratio", [1e4, 1e8, 1e14])
def test_small_values_beside_large_ones(G, orc, ratio):
    """Path rows whose values differ by `ratio`, in different channels: the
    small ones keep the accuracy of the features (bar of the other tests, per
    channel range)."""
    import torch
    T = 180
    rng = np.random.default_rng(9600)
    w = W.make_random(9600, 2, T, 1, 2, 64, 32, "f32", parent=np.stack([_broom(T, T, 40), W.random_tree(rng, T)]))
    w.S0 = np.zeros_like(w.S0)
    w.conv_w = np.zeros_like(w.conv_w)
    w.conv_w[:, 3] = 1.0  # no taps across nodes
    dep = orc.prepare(w.parent)["depth"]
    v = np.abs(w.v) + 0.5
    v[..., :16] *= np.float32(ratio) * (dep % 2 == 1)[..., None, None]
    v[..., 16:] *= (dep % 2 == 0)[..., None, None]
    w.v = v.astype(np.float32)
    print(f"[gpu] values that differ by {ratio:g}", flush=True)
    dt = G.DeviceTree(w)
    dt.prepare()
    dt.verify()
    torch.cuda.synchronize()
    ref, got = orc.verify(w), dt.out.cpu().numpy()
    for ch in (slice(0, 16), slice(16, 32)):
        err = np.max(np.abs(got[..., ch] - ref[..., ch])) / np.max(np.abs(ref[..., ch]))
        print(f"[gpu]   channels {ch.start}.. err {err:.3e}", flush=True)
        assert err <= O_TOL


@pytest.mark.parametrize("T,n", [(128, 120), (200, 180)])
def test_decays_of_either_sign(G, orc, T, n):
    """Decays below and at zero, on both sides of the on-chip size."""
    import torch
    w = W.make_random(9700, 2, T, 1, 2, 64, 32, "f32", n_valid=[n, T], shuffle=True)
    w.alpha = (w.alpha * np.random.default_rng(9700).choice([-1.0, 0.0, 1.0], w.alpha.shape, p=[0.5, 0.1, 0.4])).astype(
        np.float32)
    print(f"[gpu] decays of either sign T={T}", flush=True)
    dt = G.DeviceTree(w)
    dt.prepare()
    dt.verify()
    torch.cuda.synchronize()
    ref = orc.verify(w)
    err = np.max(np.abs(dt.out.cpu().numpy() - ref)) / np.max(np.abs(ref))
    print(f"[gpu]   err {err:.3e}", flush=True)
    assert err <= O_TOL


def test_wild_depth_in_the_metadata(G):
    """Depths by position that no tree has end the walk over deeper ancestors
    after at most T / 16 chunks; other tiles and sequences do not see them."""
    import torch
    T = 160
    w = W.make_random(9800, 2, T, 1, 2, 32, 32, "f32", parent=np.stack([W.chain_tree(T)] * 2))
    dt = G.DeviceTree(w)
    dt.prepare()
    dt.verify()
    torch.cuda.synchronize()
    clean = dt.out.clone().cpu().numpy()
    off = G.meta_layout(2, T)["pdep"]
    pdep = dt.meta[off:off + 4 * 2 * T].view(torch.int32).view(2, T)
    pdep[0, 144:] = 2 ** 31 - 1  # the last tile of the first sequence (a chain's depth-first order is its own)
    print("[gpu] wild depths in the last tile", flush=True)
    dt.verify()
    torch.cuda.synchronize()
    got = dt.out.cpu().numpy()
    np.testing.assert_array_equal(got[0, :144].view(np.int32), clean[0, :144].view(np.int32))
    np.testing.assert_array_equal(got[1].view(np.int32), clean[1].view(np.int32))


def test_rows_past_2_gb(G):
    """16640 value heads of 128 at 512 slots: the feature rows of a sequence
    span more than 2^31 bytes.  The last heads equal the same heads alone."""
    import torch
    T, dk, dv, Hv, keep = 512, 16, 128, 16640, 2
    C = 2 * dk + Hv * dv
    assert (T - 1) * 2 * C > 2 ** 31
    print(f"[gpu] rows past 2 GB: {Hv} value heads", flush=True)
    w = W.make_random(9900, 1, T, 1, keep, dk, dv, "bf16", parent=_broom(T, T, 20)[None])
    small = G.DeviceTree(w)
    small.prepare()
    small.verify()
    d = G.make_dims(1, T, 1, Hv, dk, dv, "bf16")

    def widen(x, dim, fill):
        """x as the last entries along dim of a larger tensor."""
        shape = list(x.shape)
        shape[dim] = C if x.shape[dim] == w.C else Hv
        y = torch.full(shape, fill, dtype=x.dtype, device=x.device)
        n = x.shape[dim]
        if n == w.C:  # q and k channels come first
            y.narrow(dim, 0, 2 * dk).copy_(x.narrow(dim, 0, 2 * dk))
            y.narrow(dim, C - keep * dv, keep * dv).copy_(x.narrow(dim, 2 * dk, keep * dv))
        else:
            y.narrow(dim, Hv - n, n).copy_(x)
        return y

    out = torch.empty((1, T, Hv, dv), device="cuda")
    G.verify(d, small.meta, small.q, small.k, widen(small.v, 2, 0.0), widen(small.alpha, 2, 0.5),
             widen(small.beta, 2, 0.5), widen(small.conv_w, 0, 0.0), widen(small.conv_state, 2, 0.0),
             widen(small.S0, 1, 0.0), out)
    torch.cuda.synchronize()
    assert torch.equal(out[:, :, Hv - keep:].contiguous().view(torch.int32), small.out.view(torch.int32))
    assert not out[:, :, :Hv - keep].any()


@pytest.mark.parametrize("beta", [1e-3, 1e-5, 1e-7])
def test_small_updates_of_the_query(G, orc, beta):
    """Features that fp16 holds exactly (one entry of 1, or four of 1/2): what
    is left is the walk's own error.  A weak write at node 100 gives q~ entries
    of beta / 8 that only the key of node 50, two chunks further up, reads."""
    import torch
    T, hot = 140, 30.0  # SiLU(30) = 30
    w = W.make_random(9650, 1, T, 1, 1, 32, 16, "f32", parent=W.chain_tree(T)[None])
    w.conv_w = np.zeros_like(w.conv_w)
    w.conv_w[:, 3] = 1.0  # no taps across nodes
    w.S0 = np.zeros_like(w.S0)
    w.alpha = np.ones_like(w.alpha)
    w.beta = np.full_like(w.beta, 0.5)
    w.q, w.k, w.v = np.zeros_like(w.q), np.zeros_like(w.k), np.zeros_like(w.v)
    w.q[0, :, 0, 0:4] = hot
    w.k[0, :, 0, 20] = hot
    w.k[0, 100, 0], w.k[0, 50, 0] = 0.0, 0.0
    w.k[0, 100, 0, 3:7] = hot
    w.k[0, 50, 0, 5] = hot
    w.beta[0, 100, 0] = beta
    w.v[0, 50, 0, 2] = 1024.0
    print(f"[gpu] beta = {beta:g}", flush=True)
    dt = G.DeviceTree(w)
    dt.prepare()
    dt.verify()
    torch.cuda.synchronize()
    ref, got = orc.verify(w)[0, 100:, 0, 2], dt.out.cpu().numpy()[0, 100:, 0, 2]
    assert (ref < 0).all()
    err = np.max(np.abs(got / ref - 1))
    print(f"[gpu]   err {err:.3e}", flush=True)
    # c = beta / 4 and x = c / 2 are split once or twice, off by at most 2^-38 each
    assert err <= 2.0 ** -20 + 3 * 2.0 ** -38 / (beta / 8)


@pytest.mark.parametrize("beta", [-0.5, 2.0, 3.0])
def test_writes_that_grow_the_query(G, orc, beta):
    """beta outside (0, 1], up to where q~ grows along the path."""
    import torch
    T = 180
    w = W.make_random(9660, 2, T, 1, 2, 16, 32, "f32", shuffle=True)
    w.beta[:, ::3] = beta
    print(f"[gpu] beta = {beta}", flush=True)
    dt = G.DeviceTree(w)
    dt.prepare()
    dt.verify()
    torch.cuda.synchronize()
    ref = orc.verify(w)
    err = np.max(np.abs(dt.out.cpu().numpy() - ref)) / np.max(np.abs(ref))
    print(f"[gpu]   err {err:.3e}", flush=True)
    assert err <= 2 * O_TOL  # an error is amplified as q~ is


@pytest.mark.parametrize("what", ["q", "alpha", "beta"])
@pytest.mark.parametrize("value", [float("nan"), float("inf")])
@pytest.mark.parametrize("at", [0, 7, 150])
def test_not_finite_gates_and_queries(G, orc, what, value, at):
    """The same for q and the gates of an early, a middle and a late node."""
    import torch
    T = 200
    w = W.make_random(9210 + at, 2, T, 1, 2, 32, 32, "f32", shuffle=True)
    ref = orc.prepare(w.parent)
    b = 1
    j = int(ref["order"][b, at])
    print(f"[gpu] {what} = {value} at position {at}", flush=True)
    dt = G.DeviceTree(w)
    dt.prepare()
    dt.verify()
    torch.cuda.synchronize()
    clean = dt.out.clone().cpu().numpy()
    if what == "q":
        dt.q[b, j, 0, 3] = value
    else:
        getattr(dt, what)[b, j, 1] = value
    dt.verify()
    torch.cuda.synchronize()
    got = dt.out.cpu().numpy()
    desc = np.array([i == j or (int(ref["anc"][b, i, j // 64]) >> (j % 64)) & 1 for i in range(T)], bool)
    keep = np.ones(got.shape[:3], bool)
    for h in [0, 1] if what == "q" else [1]:
        assert not np.isfinite(got[b, j, h]).all()
        keep[b, desc, h] = False
    np.testing.assert_array_equal(got[keep].view(np.int32), clean[keep].view(np.int32))
