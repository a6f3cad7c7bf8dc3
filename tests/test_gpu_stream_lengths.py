"""The rANS decoder's trips of 64 symbols: stream lengths at which its last
unbounded trip, its clamped ones and the partial one begin and end (a trip is
unbounded while 64 + 32 symbols are left), both heads.  The frame decoded from
the bitstream holds the oracle's codes at every scale: whole numbers, no
tolerance."""
import numpy as np
import pytest
import torch  # noqa: F401  (slow first import on a fresh box: at collection)

import oracle
import paper_2503_12382_amd as reno
from gpu_helpers import say, to_dev
from synth import CONFIGS, gen_weights

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("two", [False, True])
def test_streams_at_the_edges_of_trips(two, scan_cache):
    cfg = CONFIGS[0]
    B, b0 = cfg.bit_depth, cfg.min_bit_depth
    pts = scan_cache(0)
    w = gen_weights(cfg.channels, cfg.layers, seed=5, bias_std=0.1, head_scale=4.0, two_stage=two)
    P = oracle.Pyramid.from_points(pts, B, b0, cfg.range_m)
    enc, dec = (reno.Context(len(pts), B, b0, cfg.range_m, cfg.channels, cfg.layers, two_stage=two)
                for _ in range(2))
    for c in (enc, dec):
        c.set_weights(reno.weights_to_device(w))
    for L in (2, 31, 32, 33, 63, 64, 65, 95, 96, 97, 127, 128, 129, 159, 160, 161, 224):
        say("streams of", L, "two-stage" if two else "one-stage")
        dec.decode_frame(enc.encode_frame(to_dev(pts), B, stream_symbols=L).copy())
        for b in range(b0, B):
            np.testing.assert_array_equal(dec.occupancy_codes(b).cpu().numpy(), P.codes(b), err_msg=f"L={L} b={b}")
    enc.close()
    dec.close()
