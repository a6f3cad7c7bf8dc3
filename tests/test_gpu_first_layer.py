"""First conv layer (sums of cell-table rows) and the neighbour search through
the parent scale's parents, against the oracle: a one-layer model, so that the
head sees the layer alone; tile remainders, a single model scale (cells probed
directly at the base scale), the root as base, full and random occupancy codes,
both precision settings (the same kernels), and a batch of frames.

Bound: the layer sums at most 8 table rows and the bias in fp32 and the head 32
products, on sums of order 10: 1e-5 is about ten fp32 roundings of them."""
import numpy as np
import pytest
import torch  # noqa: F401  (slow first import on a fresh box: at collection)

import oracle
import paper_2503_12382_amd as reno
from gpu_helpers import say, to_dev
from synth import gen_weights

pytestmark = pytest.mark.gpu


def _cloud(n, B, R, seed, dense):
    """n distinct cells of the finest grid: a solid block, or a random surface with clumps."""
    rs = np.random.RandomState(seed)
    if dense:
        s = int(np.ceil(n ** (1 / 3)))
        g = np.stack(np.meshgrid(*[np.arange(s)] * 3, indexing="ij"), -1).reshape(-1, 3)[:n]
    else:
        g = np.unique(rs.randint(0, 1 << B, (n, 3)) // rs.choice([1, 4, 16], (n, 1)), axis=0)
    return (-R + (g + 0.5) * (2.0 * R / (1 << B))).astype(np.float32)


@pytest.mark.parametrize("n,B,b0,C,dense", [(1, 6, 4, 16, False), (15, 7, 4, 32, False), (17, 6, 4, 32, True),
                                            (64, 8, 0, 16, False), (4096, 7, 3, 32, True), (3000, 9, 4, 32, False),
                                            (70001, 10, 4, 16, False)])
@pytest.mark.parametrize("bf16x3", [False, True])
def test_one_layer_model(n, B, b0, C, dense, bf16x3):
    R = 10.0
    pts = _cloud(n, B, R, n, dense)
    w = gen_weights(C, 1, seed=n + B, bias_std=0.1)
    say("one layer", n, "points, B", B, "b0", b0, "C", C, "bf16x3", bf16x3)
    ctx = reno.Context(len(pts), B, b0, R, C, 1,
                       precision=reno.RENO_PREC_BF16X3 if bf16x3 else reno.RENO_PREC_FP32)
    ctx.set_weights(reno.weights_to_device(w))
    ctx.build_pyramid(to_dev(pts), B)
    lg = ctx.predict_probs(reno.RENO_ALL_SCALES, logits=True).cpu().numpy()
    P = oracle.Pyramid.from_points(pts, B, b0, R)
    off = 0
    for b in range(b0 + 1, B):
        ref, _, _ = P.model(b, w)
        np.testing.assert_array_equal(ctx.neighbor_map(b).cpu().numpy(), P.neighbors(b))
        err = np.abs(lg[off:off + P.num(b)] - ref).max()
        assert err <= 1e-5 * max(1.0, np.abs(ref).max()), (b, err)
        off += P.num(b)
    ctx.close()


def test_batch_of_frames_keeps_frames_apart():
    B, b0, R, C = 9, 4, 10.0, 32
    clouds = [_cloud(n, B, R, 7 + n, dense) for n, dense in ((500, False), (1, False), (729, True))]
    w = gen_weights(C, 1, seed=3, bias_std=0.1)
    say("one layer, 3 frames", [len(c) for c in clouds])
    ctx = reno.Context(sum(map(len, clouds)), B, b0, R, C, 1)
    ctx.set_weights(reno.weights_to_device(w))
    start = np.cumsum([0] + [len(c) for c in clouds]).astype(np.int64)
    ctx.build_pyramid_frames(to_dev(np.concatenate(clouds)), to_dev(start), B)
    for b in range(b0 + 1, B):
        lg = ctx.predict_probs(b, logits=True).cpu().numpy()
        ref = np.concatenate([oracle.Pyramid.from_points(c, B, b0, R).model(b, w)[0] for c in clouds])
        assert np.abs(lg - ref).max() <= 1e-5 * max(1.0, np.abs(ref).max()), b
    ctx.close()
