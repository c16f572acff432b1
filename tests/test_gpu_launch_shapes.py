"""Parity at the sizes where a kernel's launch shape or a branch of its dispatch changes.  Bars as in
tests/parity_util.py; every comparison is with the CPU oracle on the same inputs."""
import numpy as np
import pytest

import paper_2111_00705_amd as P
from oracle import oracle as O
from parity_util import STATE_RTOL, bits, make_pair, rel_close, run_steps

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


# 16-bit gradients on both sides of the line between two rows in flight and one: the fp32 entry point, which always has one,
# gives the same bits for the widened values
@pytest.mark.parametrize("n,d", [(1, 2**23 - 1), (3, 2**23 - 1), (3, 2**23), (9, 2**23), (9, 2**24 - 1), (9, 2**24)])
def test_uncompressed_16_bit_rows_in_flight(n, d):
    import torch
    print(f"[case] no compression, 16-bit gradients, d={d} n={n}", flush=True)
    gen = torch.Generator(device="cuda").manual_seed(d + n)
    for dtype, entry in ((torch.bfloat16, "step_bf16"), (torch.float16, "step_f16")):
        narrow, wide = (P.CompAms(d, n, P.TOPK, 1) for _ in range(2))
        for h in (narrow, wide):
            h.set_method(P.METHOD_NONE)
        for _ in range(2):
            g = torch.randn((n, d), device="cuda", generator=gen).to(dtype)
            getattr(narrow, entry)(g)
            wide.step(g.float())
        for name in ("get_theta", "get_m", "get_v", "get_vhat"):
            assert np.array_equal(bits(getattr(narrow, name)()), bits(getattr(wide, name)())), (name, dtype)
        narrow.destroy()
        wide.destroy()


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
            # the messages: every sign bit with its block's scale is the oracle's compressed vector (a wrong bit is off by
            # twice the scale), and so is the server's
            rows = [(i, gpu.get_scales()[i], ora.compressed[i]) for i in range(n)]
            if method == "cd":
                rows.append((n, gpu.get_server_scales(), ora.server_compressed))
            for who, scales, want in rows:
                negative = np.unpackbits(gpu.get_signs(who), bitorder="little")
                assert not negative[d:].any(), (d, n, t, who)
                spread = np.repeat(scales, B)[:d]
                assert rel_close(np.where(negative[:d], -spread, spread), want, 1e-7).all(), (d, n, t, who)
            if method == "ef":
                for i in range(n):
                    assert rel_close(gpu.get_error(i), ora.error[i], STATE_RTOL).all(), (d, n, t, i)
        for name, got, want in (("theta", gpu.get_theta(), ora.theta), ("m", gpu.get_m(), ora.m),
                                ("v", gpu.get_v(), ora.v), ("vhat", gpu.get_vhat(), ora.vhat)):
            assert rel_close(got, want, STATE_RTOL).all(), (name, d, n)
        gpu.destroy()


# bs_step_short on both sides of its lines: one to four rows of a quarter with coordinates, more workers than a wavefront has in
# flight, 64 and 65 tiles; 16-bit gradients through the same kernel are widened exactly, so both entry points agree bit for bit
@pytest.mark.parametrize("method", ["ef", "naive", "cd"])
@pytest.mark.parametrize("d,n,B", [(5, 80, 4), (1023, 80, 256), (1023, 81, 256), (1026, 40, 8), (3071, 26, 64), (3073, 20, 128),
                                   (3073, 21, 128), (64 * TILE - 3, 2, 32), (64 * TILE + 1, 2, 32)])
def test_short_blocks_in_one_launch(d, n, B, method):
    import torch
    print(f"[case] one launch, blocks of {B}, {method}, d={d} n={n}", flush=True)
    code = {"ef": (P.METHOD_EF, O.EF), "naive": (P.METHOD_NAIVE, O.NAIVE), "cd": (P.METHOD_CD, O.CD)}[method]
    handles = [P.CompAms(d, n, P.BLOCKSIGN, B) for _ in range(3)]
    ora = O.Oracle(d, n, P.BLOCKSIGN, B, 0.9, 0.999, 1e-8, 1e-3, method=code[1])
    for h in handles:
        if code[0] != P.METHOD_EF:
            h.set_method(code[0])
    gpu, b16, wide = handles
    fn = grads_of(B + d, n, d)
    for t in range(3):
        g = fn(t)
        gd = torch.from_numpy(g).cuda()
        gpu.step(gd)
        ora.step(g)
        b16.step_bf16(gd.bfloat16())
        wide.step(gd.bfloat16().float())
        assert rel_close(gpu.get_scales(), ora.scales, 1e-7).all(), t           # fp64 sums in another order
        for name, got, want in (("theta", gpu.get_theta(), ora.theta), ("m", gpu.get_m(), ora.m), ("v", gpu.get_v(), ora.v),
                                ("vhat", gpu.get_vhat(), ora.vhat)):
            assert rel_close(got, want, STATE_RTOL).all(), (name, t)
        for get in ("get_theta", "get_m", "get_v", "get_vhat", "get_scales"):
            assert np.array_equal(bits(getattr(b16, get)()), bits(getattr(wide, get)())), (get, t)
        for i in (0, n - 1):
            assert np.array_equal(b16.get_signs(i), wide.get_signs(i)), (i, t)
            negative = np.unpackbits(gpu.get_signs(i), bitorder="little")
            assert not negative[d:].any()
            spread = np.repeat(gpu.get_scales()[i], B)[:d]
            assert rel_close(np.where(negative[:d], -spread, spread), ora.compressed[i], 1e-7).all(), (i, t)
            if method == "ef":
                assert rel_close(gpu.get_error(i), ora.error[i], STATE_RTOL).all(), (i, t)
            if method == "cd":
                assert rel_close(gpu.get_ghat_worker(i), ora.ghat_workers[i], STATE_RTOL).all(), (i, t)
        if method == "cd":
            assert rel_close(gpu.get_gtilde(), ora.gtilde, STATE_RTOL).all(), t
    for h in handles:
        h.destroy()


def sparse_pair(d, n, k, method, compressor=P.TOPK):
    code = {"ef": (P.METHOD_EF, O.EF), "naive": (P.METHOD_NAIVE, O.NAIVE), "cd": (P.METHOD_CD, O.CD)}[method]
    gpu = P.CompAms(d, n, compressor, k)
    ora = O.Oracle(d, n, compressor, k, 0.9, 0.999, 1e-8, 1e-3, method=code[1])
    if code[0] != P.METHOD_EF:
        gpu.set_method(code[0])
    return gpu, ora


def selection_launches(gpu, step):
    """(kernels of the workers' selection, of the CD-Adam server's) that step() launches."""
    gpu.profile(True)
    step()
    counts = {name: launches for name, (_, launches) in gpu.profile_read().items()}
    gpu.profile(False)
    return sum(counts.get(name, 0) for name in ("tk_hist", "tk_compact", "tk_resolve")), counts.get("tk_select_server", 0)


def sparse_steps(gpu, ora, fn, steps, method, tag, dtype="float32", after=None):
    """after(t, launches): called behind each step's checks, with selection_launches of the step."""
    import torch
    step = {"float32": gpu.step, "bfloat16": gpu.step_bf16, "float16": gpu.step_f16}[dtype]
    for t in range(steps):
        g = fn(t)
        gd = torch.from_numpy(g).cuda().to(getattr(torch, dtype))
        launches = selection_launches(gpu, lambda: step(gd)) if after else step(gd)
        ora.step(g)
        for i in range(gpu.n):
            assert np.array_equal(gpu.get_selected(i)[0], ora.selected[i]), f"{tag} step {t} worker {i}: kept set"
            if method == "ef":
                assert np.array_equal(gpu.get_error(i).view(np.uint32), ora.error[i].view(np.uint32)), f"{tag} {t} {i}: error"
            if method == "cd":
                assert np.array_equal(gpu.get_ghat_worker(i).view(np.uint32), ora.ghat_workers[i].view(np.uint32)), f"{tag} {t} {i}"
        if method == "cd":
            assert np.array_equal(gpu.get_gtilde().view(np.uint32), ora.gtilde.view(np.uint32)), f"{tag} step {t}: gtilde"
        for name, got, want in (("theta", gpu.get_theta(), ora.theta), ("m", gpu.get_m(), ora.m), ("v", gpu.get_v(), ora.v),
                                ("vhat", gpu.get_vhat(), ora.vhat)):
            assert rel_close(got, want, STATE_RTOL).all(), f"{tag} step {t}: {name}"
        if after:
            after(t, launches)


# vectors of up to 16 tiles: one selection kernel, its list in registers up to 4096 entries; 17 tiles: the chain
@pytest.mark.parametrize("method", ["ef", "naive", "cd"])
@pytest.mark.parametrize("d,n,k", [(7, 1, 7), (4097, 9, 40), (16 * TILE, 2, 655), (16 * TILE, 2, 20_000), (16 * TILE + 1, 2, 655)])
def test_short_vectors(method, d, n, k):
    print(f"[case] short vectors {method} d={d} n={n} k={k}", flush=True)
    gpu, ora = sparse_pair(d, n, k, method)

    def fn(t):         # a thousandfold drop at step 3: the guess is far too high, the vector is counted anew
        return grads_of(d + k, n, d)(t) * f32(1e-3 if t == 3 else 1.0)
    sparse_steps(gpu, ora, fn, 5, method, f"{method} d={d}")
    gpu.destroy()


# a short vector whose list does not hold the k-th largest is listed again by its selection kernel, four tiles at a time:
# the first step of a handle, and every collapse of the scale under naive compression.  Part of a tile, whole tiles and
# batches of tiles, more entries than the registers hold.
@pytest.mark.parametrize("dtype", ["fp32", "bf16", "f16"])
@pytest.mark.parametrize("comp", [P.TOPK, P.RANDK])
@pytest.mark.parametrize("method", ["ef", "naive", "cd"])
def test_short_vectors_listed_again(method, comp, dtype):
    import torch
    for d, n, k in ((3, 2, 2), (4096, 2, 40), (4 * TILE + 1, 3, 170), (9 * TILE - 2, 1, 9), (16 * TILE, 2, 655), (60_001, 2, 6_001)):
        print(f"[case] short vectors listed again {method} comp={comp} {dtype} d={d} n={n} k={k}", flush=True)
        gpu, ora = sparse_pair(d, n, k, method, comp)
        tt = {"fp32": torch.float32, "bf16": torch.bfloat16, "f16": torch.float16}[dtype]
        step = {"fp32": gpu.step, "bf16": gpu.step_bf16, "f16": gpu.step_f16}[dtype]
        for t, factor in enumerate((1.0, 1.0, 2.0 ** -7, 1.0, 2.0 ** -7)):
            g = torch.from_numpy(grads_of(d, n, d)(t) * f32(100.0 * factor)).to(tt)
            step(g.cuda())
            ora.step(g.float().numpy())
            for i in range(n):
                assert np.array_equal(gpu.get_selected(i)[0], ora.selected[i]), (d, t, i)
                info = gpu.get_selection_info(i)
                if t == 0 or (factor < 1.0 and method == "naive" and comp == P.TOPK):
                    assert info["relisted"] == 1 and info["whole_bin"] != 3, (d, t, i, info)     # 3: without lists
            if method == "ef":
                assert all(np.array_equal(gpu.get_error(i).view(np.uint32), ora.error[i].view(np.uint32)) for i in range(n)), (d, t)
            if method == "cd":
                assert np.array_equal(gpu.get_server_selected()[0], ora.server_selected), (d, t)
                assert np.array_equal(gpu.get_gtilde().view(np.uint32), ora.gtilde.view(np.uint32)), (d, t)
            assert rel_close(gpu.get_theta(), ora.theta, STATE_RTOL).all(), (d, t)
        gpu.destroy()


# the same with more elements in the k-th largest's bin than the space holds (selected without lists), and with fewer
# non-zero coordinates than k
@pytest.mark.parametrize("method", ["ef", "naive", "cd"])
@pytest.mark.parametrize("share", [1.0, 0.003])
def test_short_vectors_of_equal_values_or_few_nonzeros(method, share):
    d, n, k = 60_001, 2, 600
    print(f"[case] short vectors, {share} of the coordinates equal, the others zero, {method}", flush=True)
    gpu, ora = sparse_pair(d, n, k, method)

    def fn(t):
        r = np.random.default_rng([5, t])
        return np.ascontiguousarray(np.where(r.random((n, d)) < share, f32(0.5 - 0.1 * t), f32(0.0)).astype(f32))
    sparse_steps(gpu, ora, fn, 3, method, f"{method} {share}")
    gpu.destroy()


# one launch for the selection from several regions, and three on the other side of its lines and after a miss: 32 and 64 regions (scores), the
# largest list, a scale that collapses or jumps (listed again), fewer non-zeros than k, one crowded region
@pytest.mark.parametrize("method", ["ef", "naive", "cd"])
@pytest.mark.parametrize("comp,d,n,k,kind", [
    (P.TOPK, 16 * TILE + 1, 3, 700, "plain"), (P.TOPK, 64 * TILE, 2, 14_745, "plain"), (P.TOPK, 64 * TILE + 1, 2, 2000, "plain"),
    (P.TOPK, 128 * TILE - 3, 2, 3000, "plain"), (P.TOPK, 33 * TILE, 2, 900, "collapse"), (P.TOPK, 40 * TILE - 1, 2, 900, "jump"),
    (P.TOPK, 20 * TILE + 7, 2, 900, "sparse"), (P.TOPK, 40 * TILE, 2, 1500, "crowd"), (P.TOPK, 50 * TILE, 2, 1500, "ties"),
    (P.RANDK, 513 * TILE + 9, 2, 9000, "plain"), (P.RANDK, 300 * TILE, 2, 12_000, "jump"), (P.RANDK, 20 * TILE, 2, 30, "plain")])
def test_selection_in_regions(method, comp, d, n, k, kind):
    print(f"[case] selection in regions {kind} {method} comp={comp} d={d} n={n} k={k}", flush=True)
    gpu, ora = sparse_pair(d, n, k, method, comp)
    if comp == P.RANDK:
        gpu.set_rand(3)
        ora.set_rand(3)

    def fn(t):
        x = grads_of(d + k, n, d)(t)
        r = np.random.default_rng([d, t])
        if kind == "collapse":
            x *= f32(1e-3 if t == 5 else 1.0)
        elif kind == "jump":
            x *= f32(2.0 ** 13 if t == 5 else 1.0)
        elif kind == "sparse":
            x *= (np.arange(d) % 211 == 5).astype(f32)                # about 400 coordinates that are ever non-zero
        elif kind == "crowd":
            x[:, 5 * TILE:6 * TILE] *= f32(50.0)                       # most candidates in one tile, and so in one region
        elif kind == "ties":
            x = np.where(r.random((n, d)) < 0.2, f32(1.0), x * f32(0.01)).astype(f32)
        return np.ascontiguousarray(x, dtype=f32)

    tiles, scores = (d + TILE - 1) // TILE, comp == P.RANDK
    in_rule = scores or tiles <= (128 if method == "cd" else 64)
    settled = 4 if method == "cd" and not scores else 1
    misses = []

    def after(t, launches):
        if in_rule and t >= settled and (scores or not any(misses)):
            want = 1
        else:
            want = 3
        if method == "cd" and kind != "plain" and t > 4:
            want = launches[0]                                           # the server may have missed, which no record shows
        assert want in (1, 3) and launches == (want, want if method == "cd" else 0), (t, launches)
        infos = [gpu.get_selection_info(i) for i in range(n)]
        if t >= settled and want == 1:
            misses.append(any(i["relisted"] for i in infos))
        if kind == "collapse" and t == 5 and method == "naive":
            assert all(i["relisted"] for i in infos), infos
        idx, val = gpu.get_selected(0)
        if kind == "sparse" and method == "ef":
            assert np.count_nonzero(val) < k, t                         # the threshold is a zero
        if kind == "crowd":
            assert np.count_nonzero(idx // TILE == 5) > 24 * 64 // 2, t   # more than a wavefront holds of two regions
        if kind == "ties" and method == "naive":
            assert (np.abs(val) == 1.0).all(), t                         # thousands under one value
    sparse_steps(gpu, ora, fn, 7, method, f"{kind} {method}", after=after)
    if kind in ("collapse", "jump") and method == "naive" and not scores:
        assert any(misses)
    if kind == "plain" and method != "cd":
        assert not any(misses)
    gpu.destroy()


# after a miss in one launch the selection takes three for 16 steps, for 32 where the next miss comes soon; then one again
def test_three_launches_after_a_miss_of_one_workgroup():
    d, n, k = 17 * TILE + 3, 1, 700
    print(f"[case] a collapse of the scale under naive compression, d={d}", flush=True)
    gpu, ora = sparse_pair(d, n, k, "naive")
    base = grads_of(5, n, d)(0)
    taken = []

    def fn(t):
        scale = f32(1.0 if t < 4 else 2.0 ** -3 if t < 24 else 2.0 ** -6)
        return np.ascontiguousarray(np.roll(base, 97 * t, axis=1) * scale)

    def after(t, launches):
        taken.append(launches[0])
        assert gpu.get_selection_info(0)["relisted"] == (1 if t in (0, 4, 24) else 0), t
    sparse_steps(gpu, ora, fn, 60, "naive", "collapse", after=after)
    assert taken == [3, 1, 1, 1, 1] + [3] * 16 + [1] * 4 + [3] * 32 + [1] * 3
    gpu.destroy()


# a miss sends the handle whose kernel it was to three launches, and no other; what a handle held is given back with it
def test_a_miss_is_reported_to_its_own_handle():
    import torch
    d, n, k = 17 * TILE, 1, 700
    print(f"[case] two handles, one miss, d={d}", flush=True)
    g = torch.from_numpy(grads_of(8, n, d)(0)).cuda()
    small = g * 0.125                                                    # the same order, another threshold
    for _ in range(3):
        steady, missing = (P.CompAms(d, n, P.TOPK, k) for _ in range(2))
        for h in (steady, missing):
            h.set_method(P.METHOD_NAIVE)
            for _ in range(2):
                h.step(g)
        missing.step(small)
        assert missing.get_selection_info(0)["relisted"] == 1
        taken = [selection_launches(h, lambda: h.step(x))[0] for h, x in ((steady, g), (missing, small))]
        assert taken == [1, 3]
        assert np.array_equal(missing.get_selected(0)[0], steady.get_selected(0)[0])
        steady.destroy()
        missing.destroy()


# the flags by which kernels report a miss: a handle without one takes three launches, and flags are given back
def test_more_handles_than_flags_for_misses():
    import torch
    d, n, k = 17 * TILE, 1, 700
    print(f"[case] 520 handles, d={d}", flush=True)
    g = torch.from_numpy(grads_of(8, n, d)(0)).cuda()

    def third_step(h):
        h.step(g)
        h.step(g)
        return selection_launches(h, lambda: h.step(g))[0]
    handles = [P.CompAms(d, n, P.TOPK, k) for _ in range(520)]
    taken = [third_step(handles[0]), third_step(handles[-1])]
    theta = [h.get_theta() for h in (handles[0], handles[-1])]
    assert taken == [1, 3] and np.array_equal(bits(theta[0]), bits(theta[1]))
    for h in handles:
        h.destroy()
    h = P.CompAms(d, n, P.TOPK, k)
    assert third_step(h) == 1
    h.destroy()


# CD-Adam: three launches in the steps whose guesses do not hold yet, also after the rows under the guess were replaced
def test_three_launches_until_the_markov_sequences_are_settled():
    import torch
    d, n, k = 20 * TILE, 2, 800
    print(f"[case] CD-Adam, d={d}", flush=True)
    gpu, ora = sparse_pair(d, n, k, "cd")
    fn = grads_of(6, n, d)
    taken = []
    sparse_steps(gpu, ora, fn, 7, "cd", "settling", after=lambda t, launches: taken.append(launches))
    assert taken == [(3, 3)] * 4 + [(1, 1)] * 3
    rows = np.stack([gpu.get_ghat_worker(i) for i in range(n)])
    gpu.set_markov_state(ghat_workers=rows)                              # the same numbers: the run goes on as it was
    taken = []
    for t in range(7, 13):
        g = fn(t)
        gd = torch.from_numpy(g).cuda()
        taken.append(selection_launches(gpu, lambda: gpu.step(gd)))
        ora.step(g)
        assert np.array_equal(gpu.get_gtilde().view(np.uint32), ora.gtilde.view(np.uint32)), t
    assert taken == [(3, 3)] * 4 + [(1, 1)] * 2
    gpu.destroy()


# tk_merge lists the server's candidates: its vectors loaded before the kept values up to 1023 tiles, after them beyond; a first
# step without a guess, ragged last tiles, one tile and one more than the short path takes
@pytest.mark.parametrize("comp", [P.TOPK, P.RANDK])
@pytest.mark.parametrize("d,n,k", [(1, 3, 1), (TILE - 1, 3, 200), (17 * TILE + 3, 3, 900), (1023 * TILE, 2, 5000), (1023 * TILE + 6, 2, 5000)])
def test_server_candidates_listed_by_the_merge(comp, d, n, k):
    print(f"[case] merge d={d} n={n} k={k} comp={comp}", flush=True)
    gpu, ora = sparse_pair(d, n, k, "cd", comp)
    if comp == P.RANDK:
        gpu.set_rand(9)
        ora.set_rand(9)
    sparse_steps(gpu, ora, grads_of(d, n, d), 3, "cd", f"merge {d}")
    gpu.destroy()


# tk_small_select's first digit, the fine bin above the guess: a scale that jumps 2**11 up leaves the threshold beyond the bins
# counted one by one, a dozen magnitudes leave more than 256 entries in the threshold's bin, the others a few
@pytest.mark.parametrize("method", ["ef", "naive", "cd"])
@pytest.mark.parametrize("comp", [P.TOPK, P.RANDK])
@pytest.mark.parametrize("kind", ["jump", "grid", "plain"])
def test_short_vectors_first_digit(method, comp, kind):
    d, n, k = 3 * 1024 + 5, 3, 400
    print(f"[case] first digit of a short vector, {kind}, {method}, comp={comp}", flush=True)
    gpu, ora = sparse_pair(d, n, k, method, comp)
    if comp == P.RANDK:
        gpu.set_rand(5)
        ora.set_rand(5)

    def fn(t):
        x = grads_of(17, n, d)(t) * f32(100.0)
        if kind == "grid":
            x = np.round(x * f32(64.0 / 16.0)) / f32(4.0)        # a dozen magnitudes, thousands of ties
        return np.ascontiguousarray(x * f32(2.0 ** (11 * (t % 2)) if kind == "jump" else 1.0), dtype=f32)
    sparse_steps(gpu, ora, fn, 5, method, f"{kind} {method}")
    gpu.destroy()


# tk_final_short / tk_final at the boundary between them; more than 64 kept values in a wavefront's quarter, more than
# one batch of eight workers
@pytest.mark.parametrize("tiles,n,share", [(320, 9, 0.3), (321, 9, 0.3), (320, 1, 0.001), (64, 48, 0.01), (65, 48, 0.01)])
def test_update_of_kept_values(tiles, n, share):
    d = tiles * TILE - 3
    print(f"[case] update of kept values, {tiles} tiles n={n} share={share}", flush=True)
    gpu, ora = sparse_pair(d, n, int(d * share), "ef")
    sparse_steps(gpu, ora, grads_of(tiles + n, n, d), 2, "ef", f"tiles={tiles}")
    gpu.destroy()


# the same by quarters of up to 448 tiles, and beyond; many workers with long lists on 320 tiles
@pytest.mark.parametrize("tiles,n,share", [(448, 8, 0.02), (449, 8, 0.02), (448, 1, 0.3), (448, 9, 0.01), (320, 48, 0.002), (97, 32, 0.1)])
def test_update_of_kept_values_by_quarters_of_more_tiles(tiles, n, share):
    d = tiles * TILE - 5
    k = max(1, int(share * d))
    print(f"[case] quarters of {tiles} tiles, n={n} k={k}", flush=True)
    gpu, ora = sparse_pair(d, n, k, "ef")
    sparse_steps(gpu, ora, grads_of(tiles + n, n, d), 2, "ef", f"quarters {tiles} {n}")
    gpu.destroy()


# tk_final_short: eight or five workers' kept values at a time (256 / 257 tiles), candidates beyond the two that a thread
# holds, all of a quarter kept
@pytest.mark.parametrize("comp", [P.TOPK, P.RANDK])
@pytest.mark.parametrize("tiles,n,share", [(256, 9, 0.1), (257, 11, 0.02), (17, 48, 0.3), (2, 16, 1.0), (18, 6, 0.12)])
def test_update_of_kept_values_by_quarters(tiles, n, share, comp):
    d = tiles * TILE - 5
    print(f"[case] update by quarters, {tiles} tiles n={n} share={share} comp={comp}", flush=True)
    gpu, ora = sparse_pair(d, n, int(d * share), "ef", comp)
    sparse_steps(gpu, ora, grads_of(tiles + n, n, d), 2, "ef", f"tiles={tiles}")
    gpu.destroy()


# exact ties in the threshold bin: `values` magnitudes, d / values coordinates each - ranked directly, collected in LDS
# (up to 8192 under the first digit), or scanned in place
@pytest.mark.parametrize("method", ["ef", "naive", "cd"])
@pytest.mark.parametrize("values", [2000, 60, 12])
def test_ties_in_the_threshold_bin(method, values):
    d, n = 200_003, 2
    print(f"[case] ties {method} {values} magnitudes", flush=True)
    gpu, ora = sparse_pair(d, n, 30_001, method)

    def fn(t):
        r = np.random.default_rng([values, t])
        mag = np.exp2(-r.integers(0, values, (n, d)) * (16.0 / values)).astype(f32)
        return np.ascontiguousarray(np.where(r.random((n, d)) < 0.5, mag, -mag).astype(f32))
    sparse_steps(gpu, ora, fn, 4, method, f"{method} {values}")
    gpu.destroy()


# the threshold's fine bin split by its top open bit, by index where the further bits are zero and by magnitude elsewhere:
# six magnitudes at the edges of those shares, spread over the vector or packed into few indices (more than 8192 elements
# under one digit are scanned in place, some hundred to 8192 collected in LDS)
@pytest.mark.parametrize("method", ["ef", "naive", "cd"])
@pytest.mark.parametrize("crowd,k", [("spread", 9_000), ("spread", 101), ("packed", 9_500), ("packed", 4_000), ("one value", 9_999)])
def test_split_of_the_threshold_bin(method, crowd, k):
    d, n = 4_000_003, 1                        # 22 index bits: a digit's share of the indices is 2^14
    print(f"[case] threshold bin {crowd} {method} k={k}", flush=True)
    gpu, ora = sparse_pair(d, n, k, method)
    low = np.array([0, 1, 32, 33, 0x1fff, 0x2000, 0x2001, 0x3fff], dtype=np.uint32)

    def fn(t):
        r = np.random.default_rng([k, t])
        g = (r.standard_normal((n, d), dtype=f32) * f32(1e-6))
        size = 12_000
        at = np.arange(t, t + size) if crowd == "packed" else r.choice(d, size, replace=False)
        bits = np.uint32(0x3e8000 << 8) + (low[r.integers(0, low.size, size)] if crowd == "spread" else np.where(
            r.random(size) < 0.9, np.uint32(0x2000 * (t % 2)), low[r.integers(0, low.size, size)] if crowd == "packed" else np.uint32(0x2000 * (t % 2))))
        g[0, at] = np.where(r.random(size) < 0.5, bits.astype(np.uint32).view(f32), -bits.astype(np.uint32).view(f32))
        return np.ascontiguousarray(g)
    sparse_steps(gpu, ora, fn, 3, method, f"{crowd} {k}")
    gpu.destroy()


# the same crowds as 16-bit gradients of several workers: ties at the foot of the fine bin (bfloat16) and of its upper half too
# (half precision).  The first step keeps k values of that magnitude elsewhere, which sets the guess; the second has the crowd,
# at every fourth index, so that a digit's share holds 512 of it: the k-th ends a share, or is one before or after that.
@pytest.mark.parametrize("method", ["ef", "naive", "cd"])
@pytest.mark.parametrize("dtype", ["bfloat16", "float16"])
@pytest.mark.parametrize("crowd,k", [("run", 6 * 512), ("run", 6 * 512 - 1), ("run", 6 * 512 + 1), ("one value", 5000),
                                     ("two values", 7001)])
def test_split_of_the_threshold_bin_16_bit(method, dtype, crowd, k):
    import torch
    d, n, size = 300_003, 3, 12_000            # 19 index bits: a digit's share of the indices is 2^11
    print(f"[case] threshold bin {crowd} {method} {dtype} k={k}", flush=True)
    gpu, ora = sparse_pair(d, n, k, method)
    upper = f32(1 + 2**-10) if dtype == "float16" else f32(1)         # the upper half of the fine bin that starts at 1

    def fn(t):
        r = np.random.default_rng([k, t])
        g = torch.from_numpy(r.standard_normal((n, d), dtype=f32) * f32(1e-3)).to(getattr(torch, dtype)).float().numpy()
        g[:, :150_000] = 0                                     # the crowd's: no error memory
        for i in range(n):
            if t == 0 or (t == 1 and method == "cd"):          # (CD-Adam: what was kept is subtracted)
                g[i, d - k:] = 1
            if t == 1:
                # from a share's first index on, but worker 2 from inside one
                at = 4 * np.arange(size) + (0, 2048, 1000)[i] if crowd == "run" else r.choice(150_000, size, replace=False)
                value = np.where(r.random(size) < 0.5, f32(1), upper) if crowd == "two values" else (f32(1), upper, upper)[i]
                g[i, at] = np.where(r.random(size) < 0.5, value, -value)
        return np.ascontiguousarray(g)
    for t in range(3):
        sparse_steps(gpu, ora, lambda _: fn(t), 1, method, f"{crowd} {k} step {t}", dtype)
        if t == 1:
            for i in range(n):                 # the case is what it says: listed, a fine bin that more than one share fills
                info = gpu.get_selection_info(i)
                assert info["relisted"] == 0 and info["open_bits"] == 14 and info["whole_bin"] == 0, (i, sorted(info.items()))
    gpu.destroy()


# the window of fine bins may start above the guess's coarse bin, which then is known by its count alone but listed only from the
# guess on: what lies below the guess in that bin is not kept.  A worker each: k values at fine bin 65224, k at `second` (a fall
# of 150 to 200 bins: the window starts 224 below), then `sizes` values at `bins`, then no gradient, so that the error memory is
# read again.  (A value at the foot of their coarse bin goes with the first two and is taken back: with the k values alone the
# threshold is the lower edge of the bin.)
WINDOW_CASES = {
    "k listed in the guess's bin": (65074, (64773, 64770), (4, 20)),
    "k + 1 listed in the guess's bin": (65074, (64773, 64770), (5, 20)),
    "k listed, the k-th alone in the guess's bin": (65074, (64900, 64773, 64768), (3, 1, 20)),
    "k listed, four coarse bins below the window": (65024, (64630, 64600), (4, 20)),
    "a whole bin between the guess's and the window": (65024, (64700, 64630), (4, 20)),
    "a cut in a bin between the guess's and the window": (65024, (64700, 64690), (4, 20)),
    "the guess on the edge of its bin": (65030, (64641, 64639), (4, 20)),
}


def test_threshold_below_the_window():
    d, k, n = 18 * TILE - 3728, 4, len(WINDOW_CASES)
    print(f"[case] thresholds below the window of fine bins, d={d} n={n}", flush=True)
    gpu, ora = sparse_pair(d, n, k, "ef")
    r = np.random.default_rng(5)
    guesses, foot = {}, {}

    def fn(t):
        if t == 2:
            guesses.update({i: gpu.get_selection_info(i)["next_guess"] for i in range(n)})
        g = np.zeros((n, d), dtype=f32)
        for i, (second, bins, sizes) in enumerate(WINDOW_CASES.values()):
            top = [65224, second][t] if t < 2 else 0
            fine = np.repeat(bins, sizes) if t == 2 else np.repeat(top, k if t < 2 else 0)
            at = r.choice(d, fine.size + 1, replace=False)
            low = r.integers(1, 1 << 14, fine.size)
            g[i, at[1:]] = ((fine.astype(np.uint32) << np.uint32(14)) + low.astype(np.uint32)).view(f32)
            if i in foot:
                g[i, foot[i][0]] -= foot.pop(i)[1]
            if t < 2:
                foot[i] = at[0], np.uint32((top & ~63) << 14).view(f32)
                g[i, foot[i][0]] += foot[i][1]
        return g
    for t in range(5):
        sparse_steps(gpu, ora, lambda _: fn(t), 1, "ef", f"step {t}")
        for i, name in enumerate(WINDOW_CASES):
            info = gpu.get_selection_info(i)
            if t == 2:                         # the case is what it says: listed, and only the coarse bin known at first
                assert info["relisted"] == 0 and info["open_bits"] == 20, (name, info)
                assert info["threshold_fine_bin"] >= guesses[i], (name, info, guesses[i])
    gpu.destroy()


# the same for Rand-k, whose slack is that wide where k is large: draws found on the host in which exactly k scores reach
# the guess and the k-th lies in the guess's coarse bin (worker 3 at the second step, worker 7 at the third)
@pytest.mark.parametrize("seed,n,steps", [(111, 4, 3), (63, 8, 4)])
@pytest.mark.parametrize("method", ["ef", "naive", "cd"])
def test_randk_threshold_below_the_window(method, seed, n, steps):
    d, k = 70_000, 20_000
    print(f"[case] Rand-k thresholds below the window, {method} seed={seed}", flush=True)
    gpu, ora = sparse_pair(d, n, k, method, P.RANDK)
    gpu.set_rand(seed)
    ora.set_rand(seed)
    sparse_steps(gpu, ora, grads_of(seed, n, d), steps, method, f"seed {seed}")
    gpu.destroy()


# CD-Adam on a vector long enough for more than 64 candidate regions on the server, with a drop that makes every
# selection list anew
def test_cd_lists_anew_on_a_long_vector():
    d, n = 2100 * TILE + 5, 1
    print("[case] CD-Adam lists anew, 2101 tiles", flush=True)
    gpu, ora = sparse_pair(d, n, 50_000, "cd")
    sparse_steps(gpu, ora, lambda t: grads_of(3, n, d)(t) * f32(10.0 ** (-2 * t)), 3, "cd", "long")
    gpu.destroy()


# theta asked for while the update of uniform whole-tile blocks is pending: written by the update itself to device memory
# (any 4-byte alignment, nothing past d), copied to host memory
@pytest.mark.parametrize("d", [4096, 2 * TILE + 1, 3 * TILE - 2, 5 * TILE - 1])
def test_theta_of_a_pending_update(d):
    import torch
    n = 3
    print(f"[case] theta of a pending update d={d}", flush=True)
    gpu, ora = make_pair(d, n, P.BLOCKSIGN, TILE)
    fn = grads_of(d, n, d)
    room = torch.full((d + 9,), 7.5, device="cuda")
    for t in range(4):
        g = fn(t)
        gpu.step(torch.from_numpy(g).cuda())
        ora.step(g)
        if t == 2:
            assert rel_close(gpu.get_theta(), ora.theta, STATE_RTOL).all()
        out = room[1 + t:1 + t + d]
        out.fill_(7.5)
        gpu.get_theta(out=out)
        assert rel_close(out.cpu().numpy(), ora.theta, STATE_RTOL).all(), t
        assert np.array_equal(out.cpu().numpy(), gpu.get_theta()), t
        assert bool((room[1 + t + d:] == 7.5).all()) and bool((room[:1 + t] == 7.5).all()), "written past the end"
        room.fill_(7.5)
    gpu.destroy()


# state copied to device memory by the library's own kernel (from 4 MB on; as a stream from 224 MB on): any 4-byte
# alignment, nothing past d
@pytest.mark.parametrize("d,shift", [(1 << 20, 0), ((1 << 20) + 1, 1), ((16 << 20) + 2, 3), ((16 << 20) + 4095, 2),
                                     (56 << 20, 0), ((56 << 20) + 3, 1)])
def test_large_state_to_device_memory(d, shift):
    import torch
    print(f"[case] large state to device memory d={d} shift={shift}", flush=True)
    gpu = P.CompAms(d, 1, P.TOPK, 1)
    theta = torch.randn(d, device="cuda")
    gpu.set_theta(theta)
    room = torch.full((d + 16,), 7.5, device="cuda")
    out = room[shift:shift + d]
    gpu.get_theta(out=out)
    assert torch.equal(out, theta)
    assert bool((room[:shift] == 7.5).all()) and bool((room[shift + d:] == 7.5).all())
    gpu.get_v(out=out)
    assert bool((out == 0).all())
    gpu.destroy()


# the same two ways out of the library with a destination whose allocation ends one float early: the copy that refuses it
# is the one that gets it, an error is reported, and the handle goes on
@pytest.mark.parametrize("comp,kb,d", [(P.TOPK, 1, (1 << 20) + 3), (P.BLOCKSIGN, TILE, 2 * TILE + 1)])
def test_state_to_device_memory_that_is_too_small(comp, kb, d):
    import ctypes as C
    import torch
    print(f"[case] device memory one float short, comp={comp} d={d}", flush=True)
    L = P.lib()
    gpu = P.CompAms(d, 1, comp, kb)
    theta = torch.randn(d, device="cuda")
    gpu.set_theta(theta)
    gpu.step(torch.zeros((1, d), device="cuda"))
    p = C.c_void_p()
    assert L.hipMalloc(C.byref(p), C.c_size_t(4 * (d - 1))) == 0
    getters = [L.comp_ams_get_theta, L.comp_ams_get_m, L.comp_ams_get_v, L.comp_ams_get_vhat]
    for get in getters:
        assert get(gpu._h, p, 1) == P.EDEVICE
        assert L.comp_ams_last_error(gpu._h)
    assert L.hipFree(p) == 0
    out = torch.empty(d, device="cuda")
    assert torch.equal(gpu.get_theta(out=out), theta)        # gradients of zero leave the model where it was
    gpu.destroy()
