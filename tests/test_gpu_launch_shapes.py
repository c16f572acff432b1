"""Parity at the sizes where a kernel's launch shape or a branch of its dispatch changes.  Bars as in
tests/parity_util.py; every comparison is with the CPU oracle on the same inputs."""
import numpy as np
import pytest

import paper_2111_00705_amd as P
from oracle import oracle as O
from parity_util import STATE_RTOL, make_pair, rel_close, run_steps

pytestmark = pytest.mark.gpu
f32 = np.float32
TILE = 4096


def grads_of(seed, n, d):
    def fn(t):
        r = np.random.default_rng([seed, t])
        return np.ascontiguousarray(r.standard_normal((n, d), dtype=f32) * f32(0.01))
    return fn


# bs_scale: straight from memory up to 256 pieces of a block, staged in LDS 2048 pieces at a time beyond
@pytest.mark.parametrize("pieces,ragged", [(256, 0), (257, 4095), (2048, 0), (2049, 17), (4096 + 1, 1)])
def test_block_scale_of_long_blocks(pieces, ragged):
    d = pieces * TILE - ragged
    print(f"[case] one block of {pieces} pieces, d={d}", flush=True)
    gpu, ora = make_pair(d, 1, P.BLOCKSIGN, d)
    run_steps(gpu, ora, grads_of(pieces, 1, d), 2, tag=f"pieces {pieces}", offsets=[0, d])
    gpu.destroy()


def test_block_scale_of_long_and_short_blocks_together():
    off = [0, 5, 300 * TILE + 9, 301 * TILE, 303 * TILE + 1]
    d = off[-1]
    print(f"[case] blocks of 5 coordinates to 301 pieces, d={d}", flush=True)
    gpu, ora = make_pair(d, 2, P.BLOCKSIGN, TILE, offsets=off)
    run_steps(gpu, ora, grads_of(1, 2, d), 2, tag="mixed", offsets=off)
    gpu.destroy()


# plain_update: a quarter tile per workgroup, XCD chunks from 128 tiles on
@pytest.mark.parametrize("d,n", [(1, 1), (1023, 3), (1025, 2), (127 * TILE, 2), (128 * TILE + 1, 3)])
def test_uncompressed_at_quarter_tiles(d, n):
    import torch
    print(f"[case] no compression d={d} n={n}", flush=True)
    gpu = P.CompAms(d, n, P.TOPK, 1)
    ora = O.Oracle(d, n, P.TOPK, 1, 0.9, 0.999, 1e-8, 1e-3, method=O.NONE)
    gpu.set_method(P.METHOD_NONE)
    fn = grads_of(d, n, d)
    for t in range(3):
        g = fn(t)
        gpu.step(torch.from_numpy(g).cuda())
        ora.step(g)
    for name, got, want in (("theta", gpu.get_theta(), ora.theta), ("m", gpu.get_m(), ora.m), ("v", gpu.get_v(), ora.v),
                            ("vhat", gpu.get_vhat(), ora.vhat)):
        assert rel_close(got, want, STATE_RTOL).all(), name
    gpu.destroy()


# short blocks (a power of two below a tile): butterfly sums inside a wavefront, across the wavefronts of a row, across rows;
# 3 and 1000 take the general way; d ends inside a block, a float4, a row, a tile
@pytest.mark.parametrize("B", [3, 4, 8, 16, 128, 256, 512, 1000, 1024, 2048])
@pytest.mark.parametrize("method", ["ef", "naive", "cd"])
def test_short_blocks(B, method):
    import torch
    code = {"ef": (P.METHOD_EF, O.EF), "naive": (P.METHOD_NAIVE, O.NAIVE), "cd": (P.METHOD_CD, O.CD)}[method]
    for d, n in ((B + 1, 1), (300, 20), (1024 + 255, 2), (2 * TILE, 9), (3 * TILE + 1027, 3)):
        if d <= B:
            continue
        print(f"[case] blocks of {B}, {method}, d={d} n={n}", flush=True)
        gpu = P.CompAms(d, n, P.BLOCKSIGN, B)
        ora = O.Oracle(d, n, P.BLOCKSIGN, B, 0.9, 0.999, 1e-8, 1e-3, method=code[1])
        if code[0] != P.METHOD_EF:
            gpu.set_method(code[0])
        fn = grads_of(B * 7 + d, n, d)
        for t in range(3):
            g = fn(t)
            gpu.step(torch.from_numpy(g).cuda())
            ora.step(g)
            # scales: fp64 sums of at most 2048 terms in another order differ by 1e-13 relative, fp32 keeps 6e-8
            assert rel_close(gpu.get_scales(), ora.scales, 1e-7).all(), (d, n, t)
            if method == "cd":
                assert rel_close(gpu.get_server_scales(), ora.server_scales, 1e-7).all(), (d, n, t)
            for i in range(n):
                bits = np.unpackbits(gpu.get_signs(i), bitorder="little")[:d]
                row = ora.error[i] if method == "ef" else None
                if row is not None:
                    assert rel_close(gpu.get_error(i), row, STATE_RTOL).all(), (d, n, t, i)
                assert bits.size == d
        for name, got, want in (("theta", gpu.get_theta(), ora.theta), ("m", gpu.get_m(), ora.m),
                                ("v", gpu.get_v(), ora.v), ("vhat", gpu.get_vhat(), ora.vhat)):
            assert rel_close(got, want, STATE_RTOL).all(), (name, d, n)
        gpu.destroy()
