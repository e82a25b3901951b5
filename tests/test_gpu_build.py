"""The structure build at the edges of its sorts, scans and segment tree."""
import numpy as np
import pytest

from paper_2509_07782_amd import inputs

from helpers import renderer_for

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch_cuda():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch


@pytest.mark.parametrize("bits", [4, 21])
@pytest.mark.parametrize("n", [1, 2, 3, 255, 257, 511, 512, 513, 1025, 4095, 4096, 4097, 8193, 140001])
def test_order_and_boxes(torch_cuda, n, bits):
    """Keys in stable order (4 bits an axis: thousands of equal ones) with the
    inactive Gaussians last; every child box is the union of the leaf boxes of
    its range, exactly.  n covers the one-workgroup sort (up to 4096) and the
    passes over blocks of 4096 keys, and zero to two steps of the tree."""
    rng = np.random.default_rng(n + bits)
    sc = inputs.make_scene("cluster", n, 17)
    off = rng.random(n) < 0.1
    off[0] = False
    sc["density"][off] = 0.0
    r, _ = renderer_for(sc, morton_bits=bits)
    keys, perm, aabb, nodes, _, na = r.bvh.debug()
    act = ~off & (sc["density"] > 0.01)
    assert na == act.sum()
    user = np.empty(n, np.uint64)
    user[perm] = keys
    assert np.all(user[~act] == np.uint64(1) << np.uint64(3 * bits))
    assert np.all(user[act] < np.uint64(1) << np.uint64(3 * bits))
    order = np.argsort(user, kind="stable")
    assert np.array_equal(perm, order) and np.array_equal(keys, user[order])
    mu = sc["means"][perm[:na]]
    assert np.all(aabb[:na, :3] <= mu) and np.all(aabb[:na, 3:] >= mu)
    if na < 2:
        return
    links = nodes[:na - 1][:, [3, 7]].copy().view(np.int32)
    rng_ = nodes[:na - 1][:, [11, 15]].copy().view(np.int32)
    assert np.array_equal(rng_[0], [0, na - 1])
    for c in range(2):
        link = links[:, c]
        leaf = link < 0
        inner = np.where(leaf, 0, link)
        lo = np.where(leaf, ~link, rng_[inner, 0])
        hi = np.where(leaf, ~link, rng_[inner, 1])
        # range unions: the leaves' prefix by np.minimum.reduceat over pairs
        cuts = np.stack([lo, hi + 1], 1).reshape(-1)
        ext = np.concatenate([aabb[:na], np.zeros((1, 6), np.float32)])
        mins = np.minimum.reduceat(ext[:, :3], cuts, axis=0)[::2]
        maxs = np.maximum.reduceat(ext[:, 3:], cuts, axis=0)[::2]
        box = nodes[:na - 1, 8 * c:8 * c + 8]
        assert np.array_equal(box[:, [0, 1, 2]], mins)
        assert np.array_equal(box[:, [4, 5, 6]], maxs)
    r.check_errors()
