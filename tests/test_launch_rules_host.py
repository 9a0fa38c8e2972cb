"""The rules by which the host shapes its launches (paper_2510_11400_amd/csrc/fh_rules.hpp), looked at without a GPU."""
from __future__ import annotations

import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2510_11400_amd", "csrc")


@pytest.fixture(scope="module")
def rules(tmp_path_factory):
    """rules(name, rows of integers) -> the rule's value for every row."""
    cxx = shutil.which("g++") or shutil.which("c++")
    if not cxx:
        pytest.skip("no C++ compiler")
    out = tmp_path_factory.mktemp("rules")
    src, exe = str(out / "rules.cpp"), str(out / "rules")
    with open(src, "w") as f:
        f.write('''#include "fh_rules.hpp"
#include <cstdio>
#include <cstring>
int main(int, char** argv)
{
    long long a, b, c, d;
    while (std::scanf("%lld %lld %lld %lld", &a, &b, &c, &d) == 4)
        if (!std::strcmp(argv[1], "marked_spans_per_wave")) std::printf("%lld\\n", (long long)fh::marked_spans_per_wave(a, b, c, d));
        else if (!std::strcmp(argv[1], "marked_looks_per_wave")) std::printf("%d\\n", (int)fh::marked_looks_per_wave(a, b));
        else if (!std::strcmp(argv[1], "mask_with_the_counts")) std::printf("%d\\n", (int)fh::mask_with_the_counts(a));
        else if (!std::strcmp(argv[1], "mask_with_the_counts_unranged")) std::printf("%d\\n", (int)fh::mask_with_the_counts_unranged(a, b));
        else if (!std::strcmp(argv[1], "mask_with_the_counts_apart")) std::printf("%d\\n", (int)fh::mask_with_the_counts_apart(a, b != 0, (int)c));
        else if (!std::strcmp(argv[1], "limits_apart")) std::printf("%d\\n", (int)(a < 0 ? fh::limits_apart(true, 1, (unsigned)b, (unsigned)c, d != 0) : fh::limits_apart(false, (int)a, (unsigned)b, (unsigned)c, d != 0)));
        else if (!std::strcmp(argv[1], "counters_are_crowded")) std::printf("%d\\n", (int)fh::counters_are_crowded((unsigned)a, (unsigned)b));
        else if (!std::strcmp(argv[1], "compress_in_runs")) std::printf("%d\\n", (int)fh::compress_in_runs((unsigned)a));
        else if (!std::strcmp(argv[1], "restore_in_runs")) std::printf("%d\\n", (int)fh::restore_in_runs((unsigned)a, (unsigned long long)b, (unsigned long long)c));
        else if (!std::strcmp(argv[1], "one_by_itself")) std::printf("%d\\n", (int)fh::one_by_itself((int)a, (unsigned)b));
        else if (!std::strcmp(argv[1], "maps_stay_in_cache")) std::printf("%d\\n", (int)fh::maps_stay_in_cache(a));
        else if (!std::strcmp(argv[1], "histogram_workgroups")) std::printf("%u\\n", fh::histogram_workgroups((unsigned long long)a));
        else if (!std::strcmp(argv[1], "group_sums_are_scanned")) std::printf("%d\\n", (int)fh::group_sums_are_scanned(a));
        else if (!std::strcmp(argv[1], "tile_in_run")) std::printf("%u\\n", a == 64 ? fh::tile_in_run<64>((unsigned)b, (unsigned)c) : fh::tile_in_run<128>((unsigned)b, (unsigned)c));
        else if (!std::strcmp(argv[1], "sparse_sums_are_scanned")) std::printf("%d\\n", (int)fh::sparse_sums_are_scanned((unsigned)a, (unsigned)b, (int)c));
        else if (!std::strcmp(argv[1], "decode_in_whole_lines")) std::printf("%d\\n", (int)fh::decode_in_whole_lines(a));
}
''')
    subprocess.run([cxx, "-std=c++17", "-I", CSRC, src, "-o", exe], check=True)

    def run(name, rows):
        text = "".join(" ".join(str(v) for v in r) + "\n" for r in rows)
        return [int(v) for v in subprocess.run([exe, name], input=text, text=True, check=True, capture_output=True).stdout.split()]

    return run


def test_count_pass_fills_the_device_before_a_wave_gets_a_second_span(rules):
    """Tensors of 1 to 4096 spans and beyond, one or several in a launch, beside wider ones or not: a narrow tensor's
    launch has a wave per span or at least 4096 waves' worth; a wide one's is not cut finer than 256 workgroups (of eight
    waves in its launch) ask for."""
    rows = [(n * count, n, channels, max(channels, widest)) for n in (1, 7, 255, 1024, 4095, 4096, 4097, 9000, 16384, 40000, 1 << 20)
            for count in (1, 3, 24) for channels in (1, 64, 512, 513, 768, 1024, 1025, 3072, 16384) for widest in (0, 768)]
    for (launch, tensor, channels, _), spans in zip(rows, rules("marked_spans_per_wave", rows)):
        assert 1 <= spans <= 8, (launch, tensor, channels, spans)
        if channels <= 512:
            assert spans == 1 or launch // spans >= 4096, (launch, tensor, channels, spans)
        else:
            assert spans == 1 or launch // spans >= 4096 or tensor // spans >= 2048, (launch, tensor, channels, spans)
            assert spans == 8 or tensor < 2048 * (spans + 1), (launch, tensor, channels, spans)
        assert spans == 8 or launch < 4096 * (spans + 1), (launch, tensor, channels, spans)


def test_decoder_stores_whole_lines_where_no_cache_holds_the_output(rules):
    """The memory-side cache has 256 MB: outputs well beyond it."""
    mib = 1 << 20
    rows = [(n, 0, 0, 0) for n in (0, 1, 64 * mib, 256 * mib, 384 * mib - 1, 384 * mib, 1 << 32, 26 << 32)]
    assert rules("decode_in_whole_lines", rows) == [0, 0, 0, 0, 0, 1, 1, 1]


def test_the_chains_maps_pass_the_caches_by_where_these_do_not_hold_them(rules):
    """Ordinary stores up to 96 MiB of maps in a call; from 126 MiB on they were measured to be slower."""
    mib = 1 << 20
    rows = [(n, 0, 0, 0) for n in (0, mib, 47 * 10 ** 6, 96 * mib, 96 * mib + 1, 126 * mib, 1 << 33)]
    assert rules("maps_stay_in_cache", rows) == [1, 1, 1, 1, 0, 0, 0]


def test_group_sums_are_scanned_in_launches_of_many_groups(rules):
    """Up to 4096 groups in a launch, however many streams they belong to, there is no scan."""
    assert rules("group_sums_are_scanned", [(n, 0, 0, 0) for n in (0, 1, 335, 4096, 4097, 24 * 335, 1 << 31)]) == [0, 0, 0, 0, 1, 1, 1]


def test_histogram_workgroups_of_a_stream(rules):
    """More for more symbols (a launch is sized for a bound of the count, the kernels go by the count), one for each of 256 units
    while fewer than nine vectors for a thread would take a few more, 512 at most, and their counts fit the payload's place."""
    unit = 8 * 16384
    sizes = sorted({n + d for n in (1, 65536, 1 << 22, 224 * unit, 225 * unit, 255 * unit, 256 * unit, 257 * unit, 511 * unit, 1 << 32)
                    for d in (-1, 0, 1)} | {31000000, 33000000})
    got = rules("histogram_workgroups", [(n, 0, 0, 0) for n in sizes])
    assert got == sorted(got) and got[0] == 0 and got[1] == 1 and got[-1] == 512
    of = dict(zip(sizes, got))
    assert [of[n] for n in (224 * unit - 1, 224 * unit, 31000000, 33000000, 256 * unit - 1, 256 * unit, 257 * unit)] == [256, 256, 256, 256, 256, 257, 258]
    assert [of[n] for n in (65535, 65536, 1 << 22, 511 * unit - 1, 511 * unit)] == [1, 2, 65, 511, 512]
    assert all(blocks == 1 or 1024 * blocks + 16 <= n // 8 for n, blocks in of.items() if n)


def test_sparse_sums_are_scanned_in_large_sets(rules):
    """Sets of more than 2048 groups; windows of 2 and 4 of more than 4096 while the launch has 8192 at most."""
    groups = (0, 2048, 2049, 4096, 4097, 1 << 22)
    for window in (2, 4):
        assert rules("sparse_sums_are_scanned", [(g, 8192, window, 0) for g in groups]) == [0, 0, 0, 0, 1, 1]
        assert rules("sparse_sums_are_scanned", [(g, 8193, window, 0) for g in groups]) == [0, 0, 1, 1, 1, 1]
    assert rules("sparse_sums_are_scanned", [(g, g, 8, 0) for g in groups]) == [0, 0, 1, 1, 1, 1]


def test_tiles_go_to_the_xcds_in_runs_in_large_launches_of_fp32(rules):
    tiles = (1, 8191, 8192, 12287, 12288, 1 << 31)
    rows = [(n, 0, 0, 0) for n in tiles]
    assert rules("compress_in_runs", rows) == [0, 0, 0, 0, 1, 1]
    assert rules("restore_in_runs", rows) == [0, 0, 1, 1, 1, 1]


def test_tiles_of_wide_codes_go_in_runs_in_the_largest_restores(rules):
    """Codes of 8 bits, alone or with few others, from 335 MB of fp32 on; sets of a third 8 bits, and of narrower codes, as any."""
    tiles = (8191, 8192, 40959, 40960)
    for elements, code_bits, want in ((300, 2400, [0, 0, 0, 1]), (300, 1801, [0, 0, 0, 1]), (300, 1800, [0, 1, 1, 1]), (300, 1400, [0, 1, 1, 1]),
                                      (1 << 31, 2 << 31, [0, 1, 1, 1]), (48 << 31, 8 * 48 << 31, [0, 0, 0, 1])):
        assert rules("restore_in_runs", [(n, elements, code_bits, 0) for n in tiles]) == want


@pytest.mark.parametrize("run", [64, 128])
@pytest.mark.parametrize("windows, over", [(0, 1), (0, -1), (1, -1), (1, 0), (1, 1), (3, -1), (3, 0), (3, 1), (16, 77), (24, 5)])
def test_tiles_in_runs_are_all_tiles(rules, run, windows, over):
    """Every tile once; inside a whole window every eighth workgroup has the next tile of a run, behind the last window a
    workgroup's own."""
    window = 8 * run
    blocks = windows * window + over if windows or over > 0 else window - 1
    tiles = rules("tile_in_run", [(run, b, blocks, 0) for b in range(blocks)])
    assert sorted(tiles) == list(range(blocks))
    whole = blocks // window * window
    assert tiles[whole:] == list(range(whole, blocks))
    for first in range(0, whole, window):
        for xcd in range(8):
            assert tiles[first + xcd:first + window:8] == list(range(first + xcd * run, first + (xcd + 1) * run))


def test_looks_and_masks_of_the_count_pass(rules):
    """Two looks for wide tensors of launches with a round of waves; masks with the counts for narrow ones."""
    assert rules("marked_looks_per_wave", [(n, c, 0, 0) for n in (1, 65536, 65537, 1 << 22) for c in (1, 1024, 1025, 16384)]) == [1] * 8 + [1, 1, 2, 2] * 2
    assert rules("mask_with_the_counts", [(c, 0, 0, 0) for c in (1, 1024, 1025, 16384)]) == [1, 1, 0, 0]


def test_moments_and_masks_leave_the_count_pass_in_large_launches(rules):
    """With value ranges from 8192 workgroups; without, by those that have a span for each wave: beyond 5120 of a lone tensor, from 5120
    of several, beyond 2048 where many of a tensor's meet on few counters.  The masks then come from a launch behind, except a
    lone narrow tensor's without ranges."""
    assert rules("limits_apart", [(-1, n, s, 0) for n in (1, 8191, 8192, 1 << 31) for s in (0, n)]) == [0, 0, 0, 0, 1, 1, 1, 1]
    spans = (0, 2048, 2049, 5119, 5120, 5121, 1 << 20)
    for tensors, crowded, want in ((1, 0, [0] * 5 + [1, 1]), (1, 1, [0] * 5 + [1, 1]), (2, 0, [0] * 4 + [1] * 3), (26, 1, [0, 0] + [1] * 5)):
        assert rules("limits_apart", [(tensors, 1 << 20, s, crowded) for s in spans]) == want
    rows = [(1023, 1, 0, 0), (1024, 1, 0, 0), (1024, 32, 0, 0), (1024, 33, 0, 0), (2048, 64, 0, 0), (2047, 64, 0, 0), (1 << 30, 512, 0, 0)]
    assert rules("counters_are_crowded", rows) == [0, 1, 1, 0, 1, 0, 1]
    rows = [(c, ranges, tensors, 0) for c in (1, 512, 513) for ranges in (0, 1) for tensors in (1, 2, 26)]
    assert rules("mask_with_the_counts_apart", rows) == [1, 0, 0, 0, 0, 0] * 2 + [0] * 6
    rows = [(c, spans, 0, 0) for c in (1, 512, 513, 1024, 1025) for spans in (1, 4096, 4097, 1 << 30)]
    assert rules("mask_with_the_counts_unranged", rows) == [1] * 8 + [1, 1, 0, 0] * 2 + [0] * 4


def test_short_arguments_for_one_tensor_that_the_device_holds_at_once(rules):
    assert rules("one_by_itself", [(n, tiles, 0, 0) for n in (1, 2, 26) for tiles in (1, 1792, 1793, 1 << 31)]) == [1, 1, 0, 0] + [0] * 8
