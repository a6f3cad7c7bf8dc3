"""Split-fp16 conv layers and heads (fp32 values carried as a factor and two
fp16 halves) against the oracle: magnitudes far from 1, rows and channels of
mixed magnitude, all-zero weights, the smallest and ragged tiles, and a context
whose scales are too large for 32-bit row offsets.

Bound: a product keeps 2^-22 of the row's largest entry times the channel's
largest weight, sums add in fp32: 4e-6 of the largest logit is some ten times
what three layers and a head of such sums show (2e-7 to 4e-7)."""
import numpy as np
import pytest
import torch  # noqa: F401  (slow first import on a fresh box: at collection)

import oracle
import paper_2503_12382_amd as reno
from gpu_helpers import say, to_dev
from synth import gen_weights

pytestmark = pytest.mark.gpu


def _run(pts, B, b0, R, C, L, w, two=False, max_points=None, rows=0):
    ctx = reno.Context(max_points or len(pts), B, b0, R, C, L, two_stage=two, max_model_voxels=rows)
    ctx.set_weights(reno.weights_to_device(w))
    ctx.build_pyramid(to_dev(pts), B)
    lg = ctx.predict_probs(reno.RENO_ALL_SCALES, logits=True).cpu().numpy()
    one = [ctx.predict_probs(b, logits=True).cpu().numpy() for b in range(b0 + 1, B)]
    ctx.close()
    np.testing.assert_array_equal(np.concatenate(one), lg)  # per-scale launches: the same bits
    return lg


def _check(lg, pts, B, b0, R, w, two=False, tol=4e-6):
    P = oracle.Pyramid.from_points(pts, B, b0, R)
    ref = np.concatenate([np.concatenate(P.model2(b, w)[:2], 1) if two else P.model(b, w)[0]
                          for b in range(b0 + 1, B)])
    err = np.abs(lg - ref).max() / np.abs(ref).max()
    assert err <= tol, err


def _cloud(n, B, R, seed=0):
    rs = np.random.RandomState(seed)
    g = np.stack([rs.randint(0, 1 << B, n), rs.randint(0, 1 << B, n), rs.randint(0, 1 << (B - 3), n)], 1)
    return (-R + (g + 0.5) * (2.0 * R / (1 << B))).astype(np.float32)


@pytest.mark.parametrize("scale", [1e-12, 1e-3, 1.0, 1e5, 1e12])
@pytest.mark.parametrize("C,two", [(16, False), (32, False), (32, True)])
def test_magnitudes(scale, C, two):
    """The first layer's outputs scaled far off 1, the second's scaled back, so that the split rows between them
    hold those magnitudes; head logits of order 1."""
    B, b0, R = 8, 4, 10.0
    pts = _cloud(5000, B, R, 3)
    w = gen_weights(C, 3, seed=5, bias_std=0.1, two_stage=two)
    w["conv_w"][0] = (w["conv_w"][0] * np.float32(scale)).astype(np.float32)
    w["conv_b"][0] = (w["conv_b"][0] * np.float32(scale)).astype(np.float32)
    w["conv_w"][1] = (w["conv_w"][1] / np.float32(scale)).astype(np.float32)
    say("split rows, magnitudes", scale, "C", C, "two-stage", two)
    _check(_run(pts, B, b0, R, C, 3, w, two), pts, B, b0, R, w, two)


@pytest.mark.parametrize("n", [1, 2, 15, 16, 17, 33, 255, 4097])
def test_ragged_tiles_and_mixed_channels(n):
    """Output channels of very different weight magnitude, one channel and one row's inputs all zero."""
    B, b0, R, C = 8, 3, 10.0, 32
    pts = _cloud(n, B, R, n)
    w = gen_weights(C, 3, seed=n, bias_std=0.1)
    f = (2.0 ** (np.arange(C) % 11 - 5)).astype(np.float32)  # weights stay float32
    w["conv_w"][1] = w["conv_w"][1] * f
    w["conv_b"][1] = w["conv_b"][1] * f
    w["conv_w"][2] = w["conv_w"][2] / f[:, None]
    w["conv_w"][1][:, :, 7] = 0.0
    w["conv_b"][1][7] = 0.0
    say("split rows, ragged", n)
    _check(_run(pts, B, b0, R, C, 3, w), pts, B, b0, R, w)


def test_all_zero_layer():
    B, b0, R, C = 7, 4, 10.0, 32
    pts = _cloud(700, B, R, 9)
    w = gen_weights(C, 3, seed=2, bias_std=0.1)
    w["conv_w"][1][:] = 0.0
    w["conv_b"][1][:] = 0.0
    say("split rows, zero layer")
    _check(_run(pts, B, b0, R, C, 3, w), pts, B, b0, R, w)


def test_infinite_features_stay_infinite():
    """A feature overflow (a finite weight times its count beyond fp32) reaches the logits as non-finite values, as
    in fp32 arithmetic; other voxels are untouched."""
    B, b0, R, C = 6, 4, 10.0, 32
    pts = _cloud(40, B, R, 1)
    w = gen_weights(C, 2, seed=4, bias_std=0.1)
    w["conv_b"][0][3] = np.float32(np.inf)
    say("split rows, infinite feature")
    lg = _run(pts, B, b0, R, C, 2, w)
    assert not np.isfinite(lg).any(axis=1).all() and np.isinf(lg).any()


@pytest.mark.parametrize("C,two", [(16, False), (32, False), (32, True)])
def test_context_beyond_32_bit_row_offsets(C, two):
    """max_points above 2^25 rows per scale: rows are read through 64-bit addresses; the same bits."""
    B, b0, R = 7, 4, 10.0
    pts = _cloud(9000, B, R, 6)
    w = gen_weights(C, 3, seed=8, bias_std=0.1, two_stage=two)
    say("split rows, large context", C, two)
    small = _run(pts, B, b0, R, C, 3, w, two)
    large = _run(pts, B, b0, R, C, 3, w, two, max_points=(1 << 25) + 1, rows=40000)
    np.testing.assert_array_equal(large, small)
    _check(large, pts, B, b0, R, w, two)


@pytest.mark.parametrize("C,ks,n", [(128, 3, 24000), (64, 3, 24000), (32, 5, 24000), (16, 5, 3000)])
def test_streamed_layers_staged_and_column_split(C, ks, n):
    """All scales at once stage the weights for groups of tiles (above 2048 tiles), one scale
    at a time splits each tile's columns over waves (C = 16 has one column block and never
    splits): the same bits, and the smaller scales against the oracle."""
    B, b0, R = 9, 3, 10.0
    rs = np.random.default_rng(C + ks)
    cells = np.unique(rs.integers(0, 1 << (B - 2), size=(n, 3)) + (1 << (B - 3)), axis=0)
    pts = (-10.0 + (cells + 0.5) * (20.0 / (1 << B))).astype(np.float32)
    say("streamed layers C", C, "k", ks, "points", len(pts))
    w = gen_weights(C, 2, seed=C, bias_std=0.1, two_stage=True, top=True, kernel_size=ks)
    ctx = reno.Context(len(pts), B, b0, R, C, 2, two_stage=True, top=True, kernel_size=ks)
    ctx.set_weights(reno.weights_to_device(w))
    ctx.build_pyramid(to_dev(pts), B)
    lg = ctx.predict_probs(reno.RENO_ALL_SCALES, logits=True).cpu().numpy()
    one = [ctx.predict_probs(b, logits=True).cpu().numpy() for b in range(b0 + 1, B)]
    rows = sum(ctx.num_voxels(b) for b in range(b0 + 1, B))
    ctx.close()
    assert C == 16 or rows > 16 * (2048 + B) and n <= 16 * 2048  # staged all together, split one by one
    np.testing.assert_array_equal(np.concatenate(one), lg)
    P = oracle.Pyramid.from_points(pts, B, b0, R)
    for b, got in zip((b0 + 1, b0 + 2), one):
        ref = np.concatenate(P.model2(b, w)[:2], 1)
        assert np.abs(got - ref).max() <= 4e-6 * np.abs(ref).max(), b


def _unmorton(k):
    xyz = np.zeros((len(k), 3), np.int64)
    for i in range(10):
        for ax in range(3):
            xyz[:, ax] |= ((k >> (3 * i + ax)) & 1) << i
    return xyz


@pytest.mark.parametrize("C,ks,tiles", [(128, 3, 256), (128, 3, 257), (128, 5, 1024), (128, 3, 1025), (128, 3, 2048),
                                        (128, 3, 2049), (64, 3, 512), (64, 5, 513), (64, 3, 1537), (64, 3, 2048),
                                        (32, 5, 1024), (32, 5, 1025), (32, 5, 2048)])
def test_column_split_at_the_edges_of_its_sets(C, ks, tiles):
    """A scale of exactly `tiles` tiles, alone (one to four tiles a block, one or two rounds, the last tile count
    that splits and the first that does not) and beside a full finer scale eight times its size (staged; the head's
    waves take several tiles each): the same bits.  The finer scale's rows take no part in the coarser one's sums.
    Odd counts run the one-stage head, even ones the two-stage head."""
    b, b0, R, two = 8, 6, 10.0, tiles % 2 == 0
    n = 16 * tiles - 5
    cells = _unmorton(np.arange(8 * n))  # every child of the first n cells of scale b
    B = b + 2
    pts = (-R + (2 * cells + 0.5) * (2 * R / (1 << B))).astype(np.float32)
    say("column split at", tiles, "tiles, C", C, "k", ks)
    w = gen_weights(C, 2, seed=tiles, bias_std=0.1, two_stage=two, top=True, kernel_size=ks)
    ctx = reno.Context(len(pts), B, b0, R, C, 2, two_stage=two, top=True, kernel_size=ks,
                       max_model_voxels=len(pts) * 5 // 4 + 4096)
    ctx.set_weights(reno.weights_to_device(w))
    ctx.build_pyramid(to_dev(pts), B)
    assert ctx.num_voxels(b) == n
    one = ctx.predict_probs(b, logits=True)
    lg = ctx.predict_probs(reno.RENO_ALL_SCALES, logits=True)
    first = ctx.num_voxels(b - 1)
    assert bool(torch.isfinite(one).all()) and torch.equal(lg[first:first + n], one)
    ctx.close()
