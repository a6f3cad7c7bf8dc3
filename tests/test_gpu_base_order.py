"""Base voxels out of order: the search among the sorted base keys then finds no
neighbour, not even the voxel itself, so a tile of the base scale can have no
occupied offset at all.  The frame ends in RENO_E_INPUT, and the context codes a
frame in order afterwards."""
import numpy as np
import pytest
import torch  # noqa: F401  (slow first import on a fresh box: at collection)

import oracle
import paper_2503_12382_amd as reno
from gpu_helpers import say, to_dev
from synth import gen_weights


def _search(keys, want):
    """The base search of the kernels: the last key at or below `want`, by halving, and whether it is `want`."""
    at, n = 0, len(keys)
    while n > 1:
        half = n >> 1
        at += half if keys[at + half] <= want else 0
        n -= half
    return keys[at] == want


def test_descending_keys_are_not_found():
    for n in (3, 5, 16):
        keys = list(range(n))[::-1]
        assert not any(_search(keys, k) for k in keys)
        assert all(_search(keys[::-1], k) for k in keys)
    assert not any(_search([7, 4, 1], k) for k in (7, 4, 1))


@pytest.mark.gpu
@pytest.mark.parametrize("C,ks", [(16, 5), (32, 5), (32, 3), (64, 3)])
@pytest.mark.parametrize("n", [3, 16, 400])
def test_descending_base_is_an_input_error(C, ks, n):
    B, b0 = 6, 4
    rs = np.random.default_rng(C + n)
    P = oracle.Pyramid.from_voxels(rs.integers(0, 1 << B, size=(4 * n, 3)), B, b0)
    xyz, codes = P.xyz(b0).astype(np.int32)[:n], P.codes(b0)[:n]
    w = gen_weights(C, 2, seed=C, bias_std=0.1, top=True, kernel_size=ks)
    say("descending base: C", C, "k", ks, "voxels", len(xyz))
    ctx = reno.Context(8 * P.num(B), B, b0, 10.0, C, 2, top=True, kernel_size=ks)
    ctx.set_weights(reno.weights_to_device(w))
    ctx.set_base(B, to_dev(xyz[::-1].copy()), to_dev(codes[::-1].copy()))
    ctx.expand(b0)
    ctx.predict_probs(b0 + 1)
    with pytest.raises(reno.RenoError) as e:
        ctx.sync()
    assert e.value.status == reno.RENO_E_INPUT
    ctx.set_base(B, to_dev(P.xyz(b0).astype(np.int32)), to_dev(P.codes(b0)))
    ctx.expand(b0)
    lg = ctx.predict_probs(b0 + 1, logits=True).cpu().numpy()
    ctx.sync()
    ref = P.model(b0 + 1, w)[0]
    assert np.abs(lg - ref).max() <= 1e-5 * np.abs(ref).max()  # fp32 sums of a few hundred terms of one size
    ctx.close()
