"""The contraction of unit voxels from split terms, that of edge-8 cells with
unsplit neighbours and the weight gradient of unit voxels: partial tiles, scales far from one, values that differ
by orders of magnitude between places, infinities and NaN, against the oracle."""
import numpy as np
import pytest
import torch

import octref as O
from common import U32
from paper_1611_05009_amd import octnet as oc
from paper_1611_05009_amd import synth

pytestmark = pytest.mark.gpu


def grid(p_root, p_d1, p_d2, seed, dims):
    trees = synth.random_trees(np.random.default_rng(seed), 1, *dims, p_root, p_d1, p_d2)
    return oc.from_trees(torch.from_numpy(trees.view(np.int32)).cuda(), 1, *dims), O.make_grid(trees, 1, *dims)


def cuda(a):
    return torch.from_numpy(a).cuda()


# All unit voxels (64 groups a tree), few of them (partial tiles), none.
SHAPES = [((1.0, 1.0, 1.0), (1, 1, 1)), ((1.0, 0.2, 0.1), (1, 2, 1)), ((0.1, 0.1, 0.1), (3, 3, 4)), ((0, 0, 0), (2, 3, 5)),
          ((0.5, 0.5, 0.3), (2, 3, 2))]
GROUPS = [64, 2, 0, 0, 41]  # of 8 unit voxels; a tile takes 4
PAIRS = [(32, 32), (32, 5), (16, 20), (16, 16), (8, 16), (8, 32), (4, 16), (4, 18), (64, 32)]


@pytest.mark.parametrize("cin,cout", PAIRS)
@pytest.mark.parametrize("shape", range(len(SHAPES)))
@pytest.mark.parametrize("scale", [1.0, 2.0 ** -90, 2.0 ** 60, "mixed"])
def test_scales(cin, cout, shape, scale):
    (p, dims) = SHAPES[shape]
    g, r = grid(*p, seed=shape, dims=dims)
    rng = np.random.default_rng(cin * 100 + cout)
    x = rng.standard_normal((r.n_leaves, cin)).astype(np.float32)
    w = (rng.standard_normal((cout, cin, 3, 3, 3)) / np.sqrt(27 * cin)).astype(np.float32)
    if scale == "mixed":
        x *= np.exp2(rng.integers(-12, 13, (r.n_leaves, 1))).astype(np.float32)
        w *= np.exp2(rng.integers(-6, 7, (cout, 1, 1, 1, 1))).astype(np.float32)
    else:
        x *= np.float32(scale)
    got = oc.conv3x3x3(g, torch.from_numpy(x).cuda(), torch.from_numpy(w).cuda(), impl="mfma").cpu().numpy()
    want = O.conv3(r, x, w)
    # Bound: the products of small terms left out make 1 unit of the sum of the
    # terms' magnitudes, the fp32 sums another 11 (the cells' own included).
    lim = 12 * U32 * O.conv3(r, np.abs(x), np.abs(w))
    assert (np.abs(got - want) <= lim).all(), float((np.abs(got - want) / np.maximum(lim, 1e-300)).max())


def unit_groups(r):
    """Groups of 8 unit voxels: the depth-2 bits (9 to 72) of each tree."""
    words = np.ascontiguousarray(r.trees).view(np.uint8).reshape(len(r.trees), -1)
    return int(np.unpackbits(words, axis=1, bitorder="little")[:, 9:73].sum())


def test_shapes():
    for shape, (p, dims) in enumerate(SHAPES):
        assert unit_groups(grid(*p, seed=shape, dims=dims)[1]) == GROUPS[shape]


@pytest.mark.parametrize("cin,cout", PAIRS)
@pytest.mark.parametrize("shape", [0, 3, 4])
@pytest.mark.parametrize("kind", ["row", "channels"])
def test_range(cin, cout, shape, kind):
    """No output depends on a value that its sum does not take, or on how one
    factor is shared between a channel's values and its weights."""
    (p, dims) = SHAPES[shape]
    g, r = grid(*p, seed=shape, dims=dims)
    rng = np.random.default_rng(cin * 100 + cout)
    x = rng.standard_normal((r.n_leaves, cin)).astype(np.float32)
    w = (rng.standard_normal((cout, cin, 3, 3, 3)) / np.sqrt(27 * cin)).astype(np.float32)
    if kind == "row":
        x[r.n_leaves // 2] *= np.float32(2.0 ** 40)
    else:
        f = np.exp2(rng.integers(-30, 31, cin)).astype(np.float32)
        x *= f
        w /= f.reshape(1, -1, 1, 1, 1)
    got = oc.conv3x3x3(g, torch.from_numpy(x).cuda(), torch.from_numpy(w).cuda(), impl="mfma").cpu().numpy()
    want = O.conv3(r, x, w)
    # Bound: as above.
    lim = 12 * U32 * O.conv3(r, np.abs(x), np.abs(w))
    assert (np.abs(got - want) <= lim).all(), float((np.abs(got - want) / np.maximum(lim, 1e-300)).max())


@pytest.mark.parametrize("cin,cout", [(32, 32), (16, 8), (8, 16), (4, 16)])
@pytest.mark.parametrize("shape", [0, 3])
def test_smallest_values(cin, cout, shape):
    """Values of which the last term is below bf16's normal range."""
    (p, dims) = SHAPES[shape]
    g, r = grid(*p, seed=shape, dims=dims)
    rng = np.random.default_rng(cin * 100 + cout)
    x = (rng.standard_normal((r.n_leaves, cin)) * 2.0 ** -118).astype(np.float32)
    w = rng.standard_normal((cout, cin, 3, 3, 3)).astype(np.float32)
    got = oc.conv3x3x3(g, cuda(x), cuda(w), impl="mfma").cpu().numpy()
    want = O.conv3(r, x, w)
    # Bound: as above; x is held to 2^-134 (half of bf16's smallest value),
    # the small products' sums to a few of fp32's (2^-149, 864 of them).
    ones = np.ones_like(x)
    lim = 12 * U32 * O.conv3(r, np.abs(x), np.abs(w)) + 2.0 ** -134 * O.conv3(r, ones, np.abs(w)) + 2.0 ** -139
    assert (np.abs(got - want) <= lim).all(), float((np.abs(got - want) / lim).max())


@pytest.mark.parametrize("cin,cout", [(32, 32), (16, 20), (8, 8), (4, 16)])
def test_many_tiles(cin, cout):
    """Several tiles per workgroup, the last one partial."""
    g, r = grid(1.0, 0.95, 0.95, seed=7, dims=(6, 6, 6))
    rng = np.random.default_rng(cin)
    x = rng.standard_normal((r.n_leaves, cin)).astype(np.float32)
    w = (rng.standard_normal((cout, cin, 3, 3, 3)) / np.sqrt(27 * cin)).astype(np.float32)
    b = rng.standard_normal(cout).astype(np.float32)
    got = oc.conv3x3x3(g, cuda(x), cuda(w), cuda(b), relu=True, impl="mfma").cpu().numpy()
    want = O.conv3(r, x, w, b, relu=True)
    lim = 12 * U32 * O.conv3(r, np.abs(x), np.abs(w), np.abs(b))
    assert (np.abs(got - want) <= lim).all(), float((np.abs(got - want) / lim).max())


@pytest.mark.parametrize("cin,cout", [(32, 32), (16, 8), (8, 16), (4, 16)])
@pytest.mark.parametrize("shape", [0, 3])
@pytest.mark.parametrize("bad", [np.inf, -np.inf, np.nan, 3e38])
def test_not_finite(cin, cout, shape, bad):
    (p, dims) = SHAPES[shape]
    g, r = grid(*p, seed=shape, dims=dims)
    rng = np.random.default_rng(5)
    x = rng.standard_normal((r.n_leaves, cin)).astype(np.float32)
    x[r.n_leaves // 2, cin // 2] = bad
    w = rng.standard_normal((cout, cin, 3, 3, 3)).astype(np.float32)
    with np.errstate(all="ignore"):
        want = O.conv3(r, x, w).astype(np.float32)
    got = oc.conv3x3x3(g, torch.from_numpy(x).cuda(), torch.from_numpy(w).cuda(), impl="mfma").cpu().numpy()
    fine = np.isfinite(want)
    if shape == 3 and np.isinf(bad):
        # Edge-8 cells take a row times its summed weights: infinite where
        # the oracle's sum over voxels may meet both signs.
        assert np.array_equal(np.isfinite(got), fine)
        assert np.abs(got[fine] - want[fine]).max(initial=0) <= 1e-4 * np.abs(want[fine]).max(initial=1)
    elif bad != bad or np.isinf(bad):
        assert np.array_equal(np.isnan(got), np.isnan(want))
        assert np.array_equal(got[np.isinf(want)], want[np.isinf(want)])
        assert np.abs(got[fine] - want[fine]).max(initial=0) <= 1e-4 * np.abs(want[fine]).max(initial=1)
    else:
        # Rows away from the large value keep their accuracy; the others are
        # finite wherever fp32 sums are.
        ok = fine & (np.abs(want) < 1e30)
        assert np.abs(got[ok] - want[ok]).max(initial=0) <= 1e-4 * np.abs(want[ok]).max(initial=1)
        assert np.allclose(got[fine], want[fine], rtol=1e-4, atol=1e-3)


def dw64(r, x, dy):
    return O.conv3_bwd_weight(r, x, dy)[0]


@pytest.mark.parametrize("cin,cout", [(32, 32), (32, 16), (16, 32), (16, 16)])
@pytest.mark.parametrize("shape", range(len(SHAPES)))
@pytest.mark.parametrize("scale", [1.0, 2.0 ** -60, 2.0 ** 50, "rising"])
def test_weight_gradient(cin, cout, shape, scale):
    """Unit-voxel blocks in steps that the count does not fill, and rows that
    grow along the leaf order."""
    (p, dims) = SHAPES[shape]
    g, r = grid(*p, seed=shape, dims=dims)
    rng = np.random.default_rng(cin * 100 + cout)
    x = rng.standard_normal((r.n_leaves, cin)).astype(np.float32)
    dy = rng.standard_normal((r.n_leaves, cout)).astype(np.float32)
    w = rng.standard_normal((cout, cin, 3, 3, 3)).astype(np.float32)
    if scale == "rising":
        ramp = np.exp2(np.floor(np.linspace(-30, 0, r.n_leaves)))[:, None].astype(np.float32)
        x *= ramp
        dy *= ramp[::-1] if shape % 2 else ramp
    else:
        x *= np.float32(scale)
        dy *= np.float32(scale)
    got = oc.conv3x3x3_backward(g, cuda(x), cuda(w), cuda(dy), need_input=False, need_bias=False)[1].cpu().numpy()
    want = dw64(r, x, dy)
    # Bound: fp32 products and sums, 12 units of the sum of the terms' magnitudes.
    lim = 12 * U32 * dw64(r, np.abs(x), np.abs(dy))
    assert (np.abs(got - want) <= lim).all(), float((np.abs(got - want) / np.maximum(lim, 1e-300)).max())


@pytest.mark.parametrize("cin,cout", [(32, 32), (32, 16), (16, 32), (16, 16)])
@pytest.mark.parametrize("kind", ["channels", "row", "many"])
def test_weight_gradient_range(cin, cout, kind):
    """No weight's gradient depends on values that its sum does not take: other
    channels' (by 2^60), or a row whose neighbours have no gradient; several
    blocks per workgroup."""
    g, r = grid(1.0, 1.0, 0.9, seed=3, dims=(1, 1, 4) if kind == "channels" else (6, 6, 5))
    rng = np.random.default_rng(cin * 100 + cout)
    x = rng.standard_normal((r.n_leaves, cin)).astype(np.float32)
    dy = rng.standard_normal((r.n_leaves, cout)).astype(np.float32)
    w = np.zeros((cout, cin, 3, 3, 3), np.float32)
    if kind == "row":
        x[r.prefix[1] // 2] *= np.float32(2.0 ** 40)  # of the first tree
        for t in (0, 1, 5, 6, 30, 31, 35, 36):  # it and its neighbours
            dy[r.prefix[t]:r.prefix[t + 1]] = 0
    else:
        x *= np.exp2(rng.integers(-30, 31, cin)).astype(np.float32)
        dy *= np.exp2(rng.integers(-30, 31, cout)).astype(np.float32)
    got = oc.conv3x3x3_backward(g, cuda(x), cuda(w), cuda(dy), need_input=False, need_bias=False)[1].cpu().numpy()
    want = dw64(r, x, dy)
    # Bound: as above.
    lim = 12 * U32 * dw64(r, np.abs(x), np.abs(dy))
    assert (np.abs(got - want) <= lim).all(), float((np.abs(got - want) / np.maximum(lim, 1e-300)).max())


@pytest.mark.parametrize("bad", [np.inf, np.nan, 3e38])
@pytest.mark.parametrize("side", ["x", "dy"])
def test_weight_gradient_not_finite(bad, side):
    # Unit voxels alone; the voxel (3, 3, 3) of the tree, away from its sides.
    g, r = grid(1.0, 1.0, 1.0, seed=1, dims=(1, 1, 1))
    rng = np.random.default_rng(6)
    x = rng.standard_normal((r.n_leaves, 32)).astype(np.float32)
    dy = rng.standard_normal((r.n_leaves, 16)).astype(np.float32)
    w = np.zeros((16, 32, 3, 3, 3), np.float32)
    (x if side == "x" else dy)[63, 3] = bad
    with np.errstate(all="ignore"):
        want = dw64(r, x, dy).astype(np.float32)
    got = oc.conv3x3x3_backward(g, cuda(x), cuda(w), cuda(dy), need_input=False, need_bias=False)[1].cpu().numpy()
    ok = np.isfinite(want) & (np.abs(want) < 1e30)
    assert (np.isfinite(got) == np.isfinite(want)).all()
    assert np.abs(got[ok] - want[ok]).max(initial=0) <= 1e-4 * np.abs(want[ok]).max(initial=1)
