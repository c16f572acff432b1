"""The rules that choose a launch shape from sizes (csrc/launch_rules.h), compiled by themselves on the host."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
pytestmark = pytest.mark.skipif(not shutil.which("g++"), reason="no g++")


def evaluate(tmp_path, expressions):
    """Values of C++ expressions over the header, as integers."""
    src, exe = tmp_path / "rules.cpp", tmp_path / "rules"
    lines = "\n".join(f'    std::printf("%lld\\n", (long long)({e}));' for e in expressions)
    src.write_text('#include <cstdio>\n#include "launch_rules.h"\nusing namespace cams;\nint main()\n{\n' + lines + "\n}\n")
    subprocess.run(["g++", "-std=c++17", "-Wall", "-Wextra", "-Werror", "-I",
                    os.path.join(ROOT, "paper_2111_00705_amd", "csrc"), "-o", str(exe), str(src)], check=True)
    out = subprocess.run([str(exe)], check=True, stdout=subprocess.PIPE, text=True).stdout
    return [int(x) for x in out.split()]


def test_quarter_tile_update_of_few_workers_or_few_tiles(tmp_path):
    cases = {(1, 320): 1, (1, 448): 1, (1, 449): 0, (8, 448): 1, (8, 449): 0, (9, 320): 1, (9, 321): 0, (16, 320): 1, (17, 180): 1, (24, 128): 1,
             (32, 96): 1, (48, 64): 1, (48, 320): 1, (48, 321): 0, (49, 1): 0, (64, 128): 0, (1000, 1): 0, (65535, 1): 0, (65535, 524288): 0,
             (1, 524288): 0}
    got = evaluate(tmp_path, [f"quarter_final({n}, {tiles}, false)" for n, tiles in cases])
    assert got == list(cases.values())
    naive = {(1, 448): 1, (4, 448): 1, (4, 449): 0, (5, 320): 1, (5, 321): 0, (8, 321): 0, (48, 320): 1, (49, 1): 0}
    got = evaluate(tmp_path, [f"quarter_final({n}, {tiles}, true)" for n, tiles in naive])
    assert got == list(naive.values())


def test_quarter_tile_update_holds_eight_workers_up_to_256_tiles(tmp_path):
    cases = {1: 8, 256: 8, 257: 5, 320: 5}
    got = evaluate(tmp_path, [f"short_final_batch({tiles})" for tiles in cases])
    assert got == list(cases.values())


def test_one_launch_sign_step_only_where_few_workers_share_a_quarter(tmp_path):
    cases = {(80, 1): 1, (80, 1024): 1, (81, 300): 0, (40, 1025): 1, (41, 2048): 0, (26, 2049): 1, (27, 3072): 0, (20, 3073): 1,
             (21, 3073): 0, (20, 64 * 4096): 1, (1, 64 * 4096 + 1): 0, (65535, 1): 0}
    got = evaluate(tmp_path, [f"one_launch_sign({n}, {d}, {(d + 4095) // 4096})" for n, d in cases])
    assert got == list(cases.values())


def test_one_launch_selection_of_lists_that_one_workgroup_holds(tmp_path):
    cases = {(1000, 64, 32, 0, 0): 1, (1000, 65, 32, 0, 0): 0, (1000, 128, 32, 1, 0): 1, (1000, 129, 32, 1, 0): 0, (15, 20, 32, 0, 0): 0,
             (16, 20, 32, 0, 0): 1, (18432, 60, 32, 0, 0): 1, (18433, 60, 32, 0, 0): 0, (18432, 4096, 64, 0, 1): 1,
             (18432, 4097, 64, 0, 1): 0, (18432, 4096, 128, 1, 1): 0, (1000, 20, 16, 0, 0): 0}
    calls = [f"one_launch_select({e}, {t}, {s}, {c}, {r})" for e, t, s, c, r in cases]
    assert evaluate(tmp_path, calls) == list(cases.values())


def test_the_lists_of_scores_are_priced_with_the_slack_that_one_workgroup_uses(tmp_path):
    """The k-th largest score and up, and 16 fine bins of 2**17 below it (or min_slack, where that is more): what is listed is what
    the rule compares with the 24 576 entries that the workgroup holds."""
    cases = [(1_199_882, 11_999, 6), (11_000_000, 11_000, 3), (16_700_000, 16_380, 4), (110_000_000, 11_000, 2), (110_000_000, 16_500, 2), (300_000_000, 10_000, 1),
             (1_000_000_000, 1000, 1), (70_003, 30_000, 40)]
    got = evaluate(tmp_path, [f"one_select_entries({d}, {k}, {slack}, true)" for d, k, slack in cases])
    assert got == [k + max(16, slack) * d // 2**17 for d, k, slack in cases]
    got = evaluate(tmp_path, [f"one_launch_select(one_select_entries({d}, {k}, {slack}, true), {(d + 4095) // 4096}, 64, false, true)"
                              for d, k, slack in cases])
    assert got == [1, 1, 1, 0, 0, 0, 0, 0]
    assert evaluate(tmp_path, ["one_select_entries(500000, 5000, 0, false)"]) == [6250]


def test_three_selection_launches_while_guesses_are_not_relied_on(tmp_path):
    assert evaluate(tmp_path, ["settled_steps(false)", "settled_steps(true)"]) == [1, 4]
    cases = {(0, 0): 16, (0, 10**6): 16, (16, 0): 32, (32, 255): 64, (64, 256): 16, (128, 1): 256, (256, 0): 256, (256, 300): 16}
    assert evaluate(tmp_path, [f"three_launch_steps({last}, {since})" for last, since in cases]) == list(cases.values())


def test_merge_loads_the_server_first_on_few_tiles(tmp_path):
    assert evaluate(tmp_path, [f"merge_loads_early({t})" for t in (1, 1023, 1024, 500_000)]) == [1, 1, 0, 0]


def test_candidates_of_the_largest_lists_are_stored_in_their_own_place(tmp_path):
    """From k of about 68 M on a vector's regions hold more than 2**29 entries of 8 bytes: a place counted from the first region does
    not fit a 32-bit number of bytes, the one counted from the tile's own region does."""
    checks = []
    for d, k, slices in ((2**31 - 1, 2**31 - 1, 64), (1_400_000_000, 70_000_000, 64), (600_000_007, 75_000_000, 64),
                         (600_000_007, 75_000_000, 512), (110_000_000, 110_000, 64)):
        tiles = (d + 4095) // 4096
        full = (tiles + slices - 1) // slices * 4096
        per_region = evaluate(tmp_path, [f"region_entries({d}, {k}, {full}, {slices})"])[0]
        assert per_region <= full and per_region * slices < 2**32
        if k >= 70_000_000:
            assert per_region * slices > 2**29                    # the case this is about
        assert per_region * 8 < 2**32
        for region, at in ((0, 0), (1, 0), (1, per_region - 1), (slices - 1, 0), (slices - 1, per_region - 1)):
            checks += [(vector, slices, region, per_region, at) for vector in (0, 3)]
    got = evaluate(tmp_path, [f"region_first({v}, {s}, {r}, {cap}u) * 8 + (int64_t)offset_bytes({at}, 8)" for v, s, r, cap, at in checks])
    assert got == [8 * ((v * s + r) * cap + at) for v, s, r, cap, at in checks]


def test_uncompressed_update_pads_its_grid_to_no_more_than_eight_vectors(tmp_path):
    quarters = [1, 4, 64, 511, 512, 977, 100_000, 2_097_152]
    choices = [-1, 0, 1, 16, 1024, 65_536]
    pairs = [(c, q) for c in choices for q in quarters]
    chunk = evaluate(tmp_path, [f"plain_chunk({c}, {q})" for c, q in pairs])
    grid = evaluate(tmp_path, [f"grid_blocks({q}, plain_chunk({c}, {q}))" for c, q in pairs])

    def tiles(n_blocks, ch):          # tile_of_block
        if ch <= 0:
            return list(range(n_blocks))
        span = 8 * ch
        return [b - b % span + (b % span & 7) * ch + (b % span >> 3) for b in range(n_blocks)]
    for (c, q), ch, blocks in zip(pairs, chunk, grid):
        wanted = 4 * c if c >= 0 else (64 if q >= 512 else 0)
        assert ch == min(wanted, q) and q <= blocks <= max(8 * q, q + 8 * ch)
        if q > 1000:
            continue
        # every quarter once, and on the same XCD and in the same order as with the chunk that was asked for
        order = lambda c_, n_: [(b & 7, t) for b, t in enumerate(tiles(n_, c_)) if t < q]
        asked = blocks if wanted <= 0 else (q + 8 * wanted - 1) // (8 * wanted) * 8 * wanted
        assert sorted(t for _, t in order(ch, blocks)) == list(range(q))
        assert order(ch, blocks) == order(wanted, asked)


def test_uncompressed_update_loads_two_rows_at_a_time_on_short_16_bit_vectors_alone(tmp_path):
    cases = {(1, 1, 2): 2, (8, 2**23 - 1, 2): 2, (8, 2**23, 2): 1, (9, 2**23, 2): 2, (9, 2**24 - 1, 2): 2, (9, 2**24, 2): 1,
             (32, 60_000_000, 2): 1, (1, 1, 4): 1, (16, 2**23, 4): 1, (16, 2**24, 4): 1}
    got = evaluate(tmp_path, [f"plain_rows_ahead({n}, {d}, {size})" for n, d, size in cases])
    assert got == list(cases.values())
