"""CPU checks of the launch rules and the index arithmetic that the kernels share with the host (tbe_rules.h), at sizes
that a GPU test could not take and for inputs that no kernel should be given."""
import ctypes
import os
import subprocess

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def rules(tmp_path_factory):
    so = str(tmp_path_factory.mktemp("rules") / "librules.so")
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-Wall", "-Wextra", "-Werror", "-Wno-unknown-pragmas", "-shared", "-fPIC",
                           "-I" + os.path.join(ROOT, "paper_2104_05158_amd", "csrc"),
                           os.path.join(ROOT, "tests", "rules_shim.cpp"), "-o", so])
    return ctypes.CDLL(so)


def _forward(rules, bags, lookups, wide):
    out = np.zeros(3, np.int64)
    rules.forward_launch(ctypes.c_int64(bags), ctypes.c_int64(lookups), ctypes.c_int(6), ctypes.c_int(wide),
                         out.ctypes.data_as(ctypes.c_void_p))
    return [int(x) for x in out]


@pytest.mark.parametrize("wide", [0, 1])
@pytest.mark.parametrize("bags", [1, 8191, 8192, 32767, 32768, (1 << 26) - 5, (1 << 26) - 4, (1 << 26) - 3, 1 << 26,
                                  (1 << 26) + 1, (1 << 29) - 1, 1 << 29, (1 << 31) - 1025])
def test_forward_launches_hold_every_bag_and_fit_the_grid(rules, bags, wide):
    # any number of bags a handle can be created for must be launchable: fewer than 2^32 threads
    for per_bag in (0, 5, 6, 16, 31):
        lookups = min(bags * per_bag, (1 << 31) - (1 << 24) - 1)
        one_bag, per_wave, blocks = _forward(rules, bags, lookups, wide)
        assert 1 <= per_wave <= 63
        assert blocks * 256 < 1 << 32
        assert blocks * 4 * per_wave >= bags > (blocks - 1) * 4 * per_wave
        if one_bag:
            assert per_wave == 1
        assert one_bag == int(((bags < 32768 and lookups >= 6 * bags) or (wide and lookups >= 16 * bags))
                              and bags <= (1 << 26) - 4)


def test_narrow_16_bit_rows_need_longer_bags_for_a_wavefront_each(rules):
    few = lambda epl, narrowest: rules.few_bags_lookups(ctypes.c_int(epl), ctypes.c_int(narrowest))
    assert [few(8, n) for n in range(7)] == [9, 9, 6, 6, 6, 6, 6] and [few(4, n) for n in range(7)] == [6] * 7


def test_a_call_of_any_size_has_room_for_its_buckets(rules):
    # the memory of a handle is laid out for its largest call: no smaller one may ask for more buckets
    rules.sort_buckets_max.restype = ctypes.c_int64
    most = lambda n: rules.sort_buckets_max(ctypes.c_int64(n))
    target = lambda n: rules.sort_target(ctypes.c_int64(n))
    round_of = 3584 * 704
    sizes = {1, 8193, 512 * 1024, 512 * 2560, (1 << 31) - (1 << 24) - 1} | {k * round_of for k in (1, 2, 3, 40, 800)}
    sizes = sorted(s + d for s in sizes for d in (-1, 0, 1) if s + d > 0)
    before = 0
    for n in sizes:
        t = target(n)
        assert 1024 <= t <= 3584 and before <= most(n)
        before = most(n)
        assert -(-n // t) <= most(n)
    assert target(512 * 2560) == 2560 and target(512 * 2560 + 1) == 1862 and target(round_of + 1) == 1793


@pytest.mark.parametrize("samples", [16, 1024, 8184, 8192])
@pytest.mark.parametrize("n", [8192, 20_000, (1 << 24) - 1, 1 << 24, (1 << 24) + 1, 100_000_000, (1 << 31) - (1 << 24) - 1])
def test_samples_come_from_equal_stretches_of_the_whole_table(rules, n, samples):
    got = np.empty(samples, np.int32)
    rules.sample_positions(ctypes.c_int(n), ctypes.c_int(samples), got.ctypes.data_as(ctypes.c_void_p))
    i = np.arange(samples, dtype=np.float64)
    assert np.all(got >= np.floor(i * n / samples) - 1) and np.all(got <= (i + 1) * n / samples) and np.all(got < n)


@pytest.mark.parametrize("rows", [1, 2, 5, 255, 256, 257, 70_000, (1 << 20) - 1, 1 << 20, (1 << 31) - 1])
@pytest.mark.parametrize("buckets", [1, 2, 17, 1023])
def test_every_index_finds_a_bucket_of_its_table(rules, rows, buckets):
    # borders and cells as the plan makes them; also indices that are no row of the table, such as a padding value of -1
    rng = np.random.default_rng(rows % 1000 + buckets)
    split = np.unique(np.concatenate([[0], rng.integers(0, rows, buckets - 1)])).astype(np.uint32)
    nb = len(split)
    bits = max(1, int(rows - 1).bit_length())
    lut_bits = min(12, bits, int(nb - 1).bit_length() + 3)
    shift = bits - lut_bits
    cells = np.arange((1 << lut_bits) + 1, dtype=np.int64) << shift
    lut = (np.searchsorted(split, cells, side="right") - 1).astype(np.uint16)
    inside = np.searchsorted(split, cells[1:], side="left") - 1 - lut[:-1].astype(np.int64)
    span = max(1, int(inside.max()))
    if span > 4:
        pytest.skip("bisected on the device")
    good = np.unique(np.clip(np.concatenate([split.astype(np.int64) + d for d in (-1, 0, 1)] +
                                            [rng.integers(0, rows, 1000), [rows - 1]]), 0, rows - 1))
    bad = np.array([rows, rows + 1, 1 << 31, (1 << 32) - 1, (1 << 32) - 7], np.int64)
    index = np.concatenate([good, bad]).astype(np.uint32)
    out = np.empty(len(index), np.uint32)
    below = np.concatenate([split - np.uint32(1), np.full(4, 0xffffffff, np.uint32)])
    ptr = lambda a: a.ctypes.data_as(ctypes.c_void_p)
    rules.partition_buckets(ptr(below), ptr(lut), ctypes.c_int(shift), ctypes.c_uint32((1 << lut_bits) - 1),
                            ctypes.c_int(span), ptr(index), ctypes.c_int(len(index)), ptr(out))
    assert np.array_equal(out[:len(good)], np.searchsorted(split, good, side="right") - 1)
    assert np.all(out[len(good):] < nb)


def test_a_handle_that_never_sorts_by_digits_has_no_smaller_call_that_does(rules):
    # the workspace holds the tables of the digit-by-digit sort only if the handle's largest call takes it
    use = lambda t, n, p: bool(rules.use_radix_sort(ctypes.c_int64(t), ctypes.c_int64(n), ctypes.c_int(p)))
    sizes = [1, 8192, 199_999, 200_000, 999_999, 1_000_000, 2_000_000, 3_500_000, 16_000_000, 100_000_000, 224_000_000,
             (1 << 31) - (1 << 24) - 1]
    for passes in (1, 2, 3, 4):
        for t in (1, 2, 3, 4, 8, 9, 64, 4096, 4097, 1 << 20):
            chosen = [use(t, n, passes) for n in sizes]
            assert chosen == sorted(chosen)
        assert use(4097, 1, passes)
    assert not use(64, 199_999, 1) and use(64, 200_000, 1)
    assert not use(1, 999_999, 2) and use(1, 1_000_000, 2) and not use(1, 1_999_999, 3) and use(2, 16_000_000, 3)
    assert not any(use(t, sizes[-1], 3) for t in (17, 64, 4096))


@pytest.mark.parametrize("length", [129, 130, 191, 192, 193, 255, 256, 257, 513, 5000, 128 * 256 - 1, 128 * 256, 128 * 256 + 1,
                                    128 * 255 + 1, 1_000_003, (1 << 31) - (1 << 25)])
def test_pieces_by_position_cover_a_run_and_own_their_partial_rows(rules, length):
    # rows are numbered by first position / 64: no piece may be shorter, or the next one (of this run or of the one behind
    # it) could have the same row
    for s in (0, 1, 63, 127, 128, 1_000_001):
        out = np.empty(257, np.int32)
        np_ = rules.position_pieces(ctypes.c_int(s), ctypes.c_int(length), out.ctypes.data_as(ctypes.c_void_p))
        borders = out[:np_ + 1].astype(np.int64)
        sizes = np.diff(borders)
        assert borders[0] == s and borders[-1] == s + length and np_ <= 256
        assert sizes.min() >= 64 and sizes.max() - sizes.min() <= 1
        assert sizes.max() <= 128 or np_ == 256
        assert len(np.unique(borders // 64)) == np_ + 1


def test_every_piece_starts_at_one_row_of_partial_sums(rules):
    # what a wavefront finds that looks at the 64 positions of a partial row: the piece that starts there, if any
    for s, length in [(0, 129), (63, 129), (64, 129), (1, 256), (77, 257), (130, 1000), (5, 32768), (5, 32769), (9, 32767 + 256), (127, 100_003)]:
        out = np.empty(257, np.int32)
        np_ = rules.position_pieces(ctypes.c_int(s), ctypes.c_int(length), out.ctypes.data_as(ctypes.c_void_p))
        starts = out[:np_].tolist()
        found = {}
        for slot in range(s // 64, (s + length - 1) // 64 + 1):
            i = rules.first_piece_from(ctypes.c_int(length), ctypes.c_int(np_), ctypes.c_int(slot * 64 - s))
            assert i == next((j for j, p in enumerate(starts) if p >= slot * 64), np_)
            if i < np_ and starts[i] < slot * 64 + 64:
                found[i] = slot
        assert found == {i: p // 64 for i, p in enumerate(starts)}


def test_which_long_runs_are_cut_how(rules):
    def rule(n, batch, widest, grad_bytes):
        out = np.empty(4, np.int32)
        rules.long_run_rule(ctypes.c_int64(n), ctypes.c_int64(batch), ctypes.c_int64(widest), ctypes.c_int(grad_bytes),
                            out.ctypes.data_as(ctypes.c_void_p))
        return out[:3].tolist()
    def found(n, batch):
        out = np.empty(4, np.int32)
        rules.long_run_rule(ctypes.c_int64(n), ctypes.c_int64(batch), ctypes.c_int64(128), ctypes.c_int(4), out.ctypes.data_as(ctypes.c_void_p))
        return bool(out[3])
    assert found(1 << 19, 8192) and not found((1 << 19) + 1, 8192) and not found(1000, 8193)
    assert rule(3_999_999, 8192, 128, 4) == [1, 0, 128] and rule(4_000_000, 8192, 128, 4) == [1, 1, 512]
    assert rule(4_000_000, 8193, 128, 4) == rule(1, 8193, 128, 4) == [0, 1, 512] and rule(1, 8193, 128, 2) == [1, 0, 128]
    assert rule(8_388_607, 2048, 512, 4) == [1, 0, 128] and rule(8_388_608, 2048, 512, 4) == [1, 1, 512]
    assert rule(7_999_999, 8193, 128, 2) == [1, 0, 128] and rule(8_000_000, 8193, 128, 2) == [1, 1, 512]


def test_spans_shorten_while_the_chip_has_room_for_more_wavefronts(rules):
    span = lambda n, lanes, tables: rules.update_span(ctypes.c_int64(n), ctypes.c_int64(lanes), ctypes.c_int64(tables))
    assert [span(n, 1, 1) for n in (1, 65_536, 65_537, 131_072, 131_073, 262_144, 262_145)] == [16, 16, 32, 32, 64, 64, 128]
    assert span(1_048_576, 16 * 7, 7) == 16 and span(1_048_577, 16 * 7, 7) == 32
    assert span((1 << 31) - (1 << 24), 64 << 20, 1 << 20) == 128


def test_which_calls_have_units_that_find_their_lookups_themselves(rules):
    use = lambda t, n: bool(rules.use_select_sort(ctypes.c_int64(t), ctypes.c_int64(n)))
    assert use(1, 24_576) and not use(1, 24_577) and use(10, 245_760) and not use(10, 245_761)
    assert use(11, 1 << 18) and use(4096, 1 << 18) and not use(4096, (1 << 18) + 1)


def test_hot_rows_take_no_more_units_than_there_is_room_for(rules):
    # whatever rows a table's samples are of: the units beyond one each are at most one per 4096 lookups
    rng = np.random.default_rng(11)
    parts = lambda sampled, n, samples: rules.select_parts(ctypes.c_int(sampled), ctypes.c_int(n), ctypes.c_int(samples))
    for n in (1025, 4095, 4096, 8191, 8192, 100_003, (1 << 18) - 1, 1 << 18):
        want = (n + 1023) // 1024
        samples = want * min(16, 8192 // want)
        assert parts(samples, n, samples) == 1 + n // 4096
        cuts = np.sort(rng.integers(0, samples + 1, 40))
        of_rows = np.diff(np.concatenate([[0], cuts, [samples]]))
        assert sum(parts(int(k), n, samples) - 1 for k in of_rows) <= n // 4096


def test_which_calls_have_units_that_collect_their_pieces(rules):
    # a chunk is put in order by one workgroup at once, a unit holds the starts of all chunks and shifts by their length: a chunk
    # of more than a tile, or of no power of two, may never take that path, whatever the host asks for
    use = lambda words32, n, chunk: bool(rules.use_pieces_sort(ctypes.c_int(words32), ctypes.c_int64(n), ctypes.c_int(chunk)))
    for chunk in (2048, 4096, 8192):
        assert use(1, 24_577, chunk) and use(1, 1024 * chunk, chunk) and not use(1, 1024 * chunk + 1, chunk) and not use(0, 1024 * chunk, chunk)
    for chunk in (8193, 16_384, 24_576, 32_768, 6144, 5000):
        assert not use(1, 1_000_000, chunk) and not use(1, 1 << 24, chunk), chunk


def test_every_unit_of_the_bucket_sort_has_a_workgroup_or_takes_a_ticket(rules):
    rules.sort_local_blocks.restype = ctypes.c_int64
    blocks = lambda n, tables, target: rules.sort_local_blocks(ctypes.c_int64(n), ctypes.c_int64(tables), ctypes.c_int(target),
                                                               ctypes.c_int(8192), ctypes.c_int64(768))
    assert blocks(32_769, 1, 1024) == 768                # no fewer than are resident
    assert blocks(8_000_000, 1, 2841) == 2815 + 976 + 2  # a unit per bucket, one more per tile of a row, two a table
    assert blocks(100_000, 4000, 1024) == 97 + 12 + 8000 and blocks(100_000, 4041, 1024) == 8191 and blocks(100_000, 4042, 1024) == 768
    assert blocks(100_000_000, 64, 3500) == 768


def test_rows_of_several_units_fit_the_units_of_their_call(rules):
    # the plan of a call of up to 8 M lookups takes part numbers from the samples: whatever rows those are of, at most one unit
    # more for every tile of lookups
    rng = np.random.default_rng(12)
    parts = lambda sampled, n, samples: rules.unit_parts(ctypes.c_int(sampled), ctypes.c_int(n), ctypes.c_int(samples), ctypes.c_int(8192))
    for n in (32_769, 131_073, 786_433, 4_000_003, (1 << 23) - 1, 1 << 23):
        for samples in (16, 1000, 8192):
            assert parts(samples, n, samples) == 1 + n // 8192
            cuts = np.sort(rng.integers(0, samples + 1, 40))
            of_rows = np.diff(np.concatenate([[0], cuts, [samples]]))
            assert sum(parts(int(k), n, samples) - 1 for k in of_rows) <= n // 8192


def _parts_of_a_unit(rules, looked_up, rows):
    """What sort_select_kernel does with a unit of `rows` rows: its parts as (first row, rows, lookups), and the walks."""
    rules.select_fewer_rows.restype = rules.select_next_rows.restype = ctypes.c_uint32
    at = np.sort(looked_up)
    lo, size, walks, done, parts, total = 0, rows, 0, 0, [], None
    while lo < rows:
        m = int(np.searchsorted(at, lo + size) - np.searchsorted(at, lo))
        walks += 1
        total = m if total is None else total
        if m > 6144 and size > 1:
            size = rules.select_fewer_rows(ctypes.c_uint32(size), ctypes.c_int(m))
            continue
        parts.append((lo, size, m))
        done += m
        lo += size
        if done == total:
            break
        size = rules.select_next_rows(ctypes.c_uint32(size), ctypes.c_int(m), ctypes.c_uint32(rows - lo), ctypes.c_int(total - done))
    return parts, walks


@pytest.mark.parametrize("rows", [2, 3, 7000, 1_000_000, (1 << 32) - 1])
def test_a_unit_that_does_not_fit_is_cut_into_few_parts(rules, rows):
    rng = np.random.default_rng(rows % 977)
    n, few = 200_000, min(rows, 1000)
    for looked_up in (rng.integers(0, few, n), rng.integers(rows - few, rows, n), rng.integers(0, rows, n), rng.integers(0, rows, 6145),
                      rng.choice(min(rows, 1 << 20), few, replace=False)[rng.integers(0, few, n)],
                      (rows * 2.0 ** -rng.integers(0, 33, n) * rng.random(n)).astype(np.int64),
                      np.concatenate([np.full(7000, rows // 3), rng.integers(0, rows, 5000)])):
        looked_up = np.minimum(looked_up, rows - 1)
        parts, walks = _parts_of_a_unit(rules, looked_up, rows)
        assert all(m <= 6144 or size == 1 for _, size, m in parts) and sum(m for *_, m in parts) == looked_up.size
        assert all(a + size == b for (a, size, _), (b, *_) in zip(parts, parts[1:])) and parts[0][0] == 0
        # down and up the rows once, and two walks a part
        assert walks <= 2 * np.log2(rows) + 2 * (looked_up.size / 6144 + 1)


def test_small_calls_sum_their_long_runs_in_at_most_32_trips(rules):
    small = lambda n, lanes: bool(rules.small_long_runs(ctypes.c_int64(n), ctypes.c_int(lanes)))
    assert small(512, 64) and not small(513, 64) and small(4096, 8) and not small(4097, 8) and small(8192, 4) and small(8192, 1)
