"""Decoded codes whose children exceed a scale's capacity: every stored (code,
first child) names rows of the scale only, so the launches that follow stay
inside their buffers, and the frame ends in RENO_E_CAPACITY."""
import ctypes
import os
import shutil
import subprocess

import numpy as np
import pytest
import torch  # noqa: F401  (slow first import on a fresh box: at collection)

import oracle
import paper_2503_12382_amd as reno
from gpu_helpers import say, to_dev
from paper_2503_12382_amd import build as hip_build
from synth import gen_weights


@pytest.mark.skipif(not (os.path.exists("/opt/rocm/bin/hipcc") or shutil.which("hipcc")), reason="no hipcc")
def test_kept_children_are_the_lowest_that_fit(tmp_path):
    """The rule of the expansion kernel, on the host, for every code and every number of rows left."""
    src, so = tmp_path / "kept.cpp", tmp_path / "kept.so"
    src.write_text(f'#include "{hip_build.CSRC}/dev.h"\n'
                   'extern "C" unsigned kept(unsigned c, long long f, long long cap) '
                   '{ return reno::kept_children(c, f, cap); }\n')
    subprocess.run([hip_build.hipcc(), "-x", "hip", "--cuda-host-only", "-O1", "-std=c++17", "-shared", "-fPIC",
                    str(src), "-o", str(so)], check=True, capture_output=True)
    kept = ctypes.CDLL(str(so)).kept
    kept.argtypes = [ctypes.c_uint, ctypes.c_longlong, ctypes.c_longlong]
    for cap in (0, 1, 7, 8, 1000, (1 << 30) - 1):
        for room in range(-9, 12):
            for code in range(256):
                bits = [d for d in range(8) if code >> d & 1][:max(room, 0)]
                assert kept(code, cap - room, cap) == sum(1 << d for d in bits), (cap, room, code)


@pytest.mark.gpu
@pytest.mark.parametrize("C,ks,top,two", [(16, 3, False, False), (32, 3, False, True), (32, 3, True, False),
                                          (16, 5, True, True), (64, 3, True, False)])
def test_dense_codes_beyond_the_capacity(C, ks, top, two):
    """Full codes from scale 2 on in a context of 3001 voxels a scale: scale 4 and every later one is cut off."""
    B, b0, cap = 9, 2, 3001
    w = gen_weights(C, 2, seed=C + ks, bias_std=0.1, two_stage=two, top=top, kernel_size=ks)
    say("codes beyond the capacity: C", C, "k", ks, "full predictor", top, "two-stage", two)
    ctx = reno.Context(cap, B, b0, 10.0, C, 2, two_stage=two, top=top, kernel_size=ks)
    ctx.set_weights(reno.weights_to_device(w))

    def decode(base, codes):
        ctx.set_base(B, to_dev(base.astype(np.int32)), to_dev(codes[b0]))
        for b in range(b0 + 1, B):
            ctx.expand(b - 1, None if b - 1 == b0 else to_dev(codes[b - 1]))
            ctx.predict_probs(b)
            if two:
                ctx.predict_second(b, to_dev(codes[b] & 15))
        ctx.expand(B - 1, to_dev(codes[B - 1]))

    full = oracle.Pyramid.from_voxels(np.stack(np.meshgrid(*[np.arange(4)] * 3, indexing="ij"), -1).reshape(-1, 3),
                                      b0, 0)
    decode(full.xyz(b0), {b: np.full(64 if b == b0 else cap, 255, np.uint8) for b in range(b0, B)})
    with pytest.raises(reno.RenoError) as e:
        ctx.sync()
    assert e.value.status == reno.RENO_E_CAPACITY
    # the context codes a frame that fits afterwards
    rs = np.random.default_rng(C)
    P = oracle.Pyramid.from_voxels(rs.integers(0, 1 << B, size=(400, 3)), B, b0)
    decode(P.xyz(b0), {b: P.codes(b) for b in range(b0, B)})
    np.testing.assert_array_equal(ctx.coords(B)[1].cpu().numpy().view(np.uint64), P.keys(B))
    bits, _ = ctx.code_length(reno.RENO_ALL_SCALES)
    ref = np.concatenate([(P.model2(b, w)[4] if two else P.model(b, w)[2]) for b in range(b0 + 1, B)])
    assert np.abs(bits.cpu().numpy() - ref).max() <= 1e-4  # fp32 logits of order 10, rounded some hundred times
    ctx.close()
