"""[B, n, D] with columns of channels that do not fill the lanes (whole narrow items, or 64 channels whatever item
they belong to), rows that do not keep to 128-byte lines with few and many tiles, and few columns of many tiles:
two carry levels of eight or sixteen, whose records the waves of a tile share."""
import numpy as np
import pytest

import oracle
from paper_2311_06281_amd import workloads

import test_gpu_cross_product as cross
from test_gpu_cross_product import gpu  # noqa: F401  (fixture)

pytestmark = pytest.mark.gpu

# (B, n, D)
SHAPES = [
    (2, 300, 96), (3, 700, 65), (5, 65, 33), (4, 129, 100), (2, 33, 48), (7, 1100, 40), (3, 257, 1000 - 25),  # dense columns
    (130, 2100, 33), (8, 1100, 96),                                                                            # the same, several tiles
    (9, 513, 19), (13, 70, 5), (3, 300, 31), (6, 2000, 21),                                                    # whole items
    (4, 16001, 70), (2, 100003, 20), (70, 3000, 13), (40, 2900, 37),
    # few columns: one tile more than a group (8 tiles of 256 steps), than a super-group (64), than several
    (1, 1025, 64), (1, 2049, 66), (2, 256 * 9 + 3, 96), (1, 256 * 64 + 1, 128), (1, 256 * 65, 2), (3, 256 * 72 + 5, 65),
    (9, 256 * 8 + 1, 64), (12, 256 * 16, 64), (15, 256 * 24, 64), (100, 256 * 4 + 9, 64),  # groups of eight, uneven queues
    (2, 256 * 200 + 77, 48), (1, 256 * 512, 5), (15, 256 * 17, 64), (14, 256 * 16 + 255, 64),
]


@pytest.mark.parametrize("mode", list(cross.MODES))
@pytest.mark.parametrize("bf16", [False, True])
def test_columns_and_carry_levels(gpu, mode, bf16):
    rng = np.random.default_rng(sum(map(ord, mode)) + 7 * int(bf16))
    for shape in SHAPES:
        a, b, x0 = cross._inputs(rng, shape, "BND", mode)
        if bf16:  # the bf16-rounded values are what is stored: they define the problem
            a = workloads.bf16_bits_to_f32(workloads.f32_to_bf16_bits(a)).reshape(a.shape)
            b = workloads.bf16_bits_to_f32(workloads.f32_to_bf16_bits(b)).reshape(b.shape)
        for offset in (0, 1):
            print(f"[columns] {mode} bf16={bf16} shape={shape} offset={offset}", flush=True)
            got = cross._run(gpu, a, b, x0, "BND", cross.MODES[mode], bf16, offset_elems=offset)
            cross._check(got, a, b, x0, "BND", mode)


# Few columns of tall tiles (sixteen waves, 512 steps; two carry levels of sixteen): just enough tiles, the last one a step long or
# missing one, a group and one tile more, a super-group (256 tiles) and one tile more, whole items in their lanes and as runs,
# columns of channels of two items, the most columns of
# few.  One round of more columns; two rounds of columns that cut lines, and as runs.
@pytest.mark.parametrize("mode", ["signed", "log_logout", "positive"])
@pytest.mark.parametrize("bf16", [False, True])
@pytest.mark.parametrize("shape", [
    (1, 512 * 128 + 1, 64), (1, 512 * 129 - 1, 64), (8, 512 * 17, 64), (8, 512 * 16 + 33, 64), (1, 512 * 256 + 1, 70), (1, 512 * 257, 33),
    (3, 512 * 90 + 31, 96), (16, 512 * 16 + 5, 64), (24, 512 * 21, 64), (32, 512 * 8, 64), (5, 512 * 130 + 7, 32), (40, 512 * 45 + 3, 5), (9, 512 * 70 + 1, 30),
    (3, 512 * 6 - 5, 769), (16, 512 * 4, 256), (4, 512 * 5 - 511, 768), (5, 512 * 9 - 31, 611), (124, 512 * 15 + 1, 16), (154, 512 * 5 - 9, 16), (60, 512 * 65 + 7, 2), (611, 512 * 10 - 2, 2),
])
def test_tall_tiles(gpu, mode, bf16, shape):
    torch, hb = gpu
    B, n, D = shape
    flags = hb.flags_from_names(cross.MODES[mode]) | (hb.HEINSEN_IN_BF16 if bf16 else 0)
    tall = n > 512 * 14 or (D % 32 == 0 or n > 512 * 8) or not bf16  # one round of bf16 that cuts lines keeps the small ones
    assert hb.heinsen_tile_shape(B, D, n, hb.HEINSEN_LAYOUT_BND, flags)[1] == (512 if tall and not (bf16 and B == 124) else 256)
    rng = np.random.default_rng(sum(shape) + int(bf16))
    a, b, x0 = cross._inputs(rng, shape, "BND", mode)
    if bf16:  # the bf16-rounded values are what is stored: they define the problem
        a = workloads.bf16_bits_to_f32(workloads.f32_to_bf16_bits(a)).reshape(a.shape)
        b = workloads.bf16_bits_to_f32(workloads.f32_to_bf16_bits(b)).reshape(b.shape)
    print(f"[tall] {mode} bf16={bf16} shape={shape}", flush=True)
    got = cross._run(gpu, a, b, x0, "BND", cross.MODES[mode], bf16, offset_elems=0)
    cross._check(got, a, b, x0, "BND", mode)
    for _ in range(3):  # whatever order the records come in
        again = cross._run(gpu, a, b, x0, "BND", cross.MODES[mode], bf16, offset_elems=0)
        assert np.array_equal(got.view(np.uint32), again.view(np.uint32))


# Two carry levels, a tile whose summary never comes: its column is NaN from the next tile on, the others are as they were.
@pytest.mark.parametrize("shape,drop", [((2, 256 * 70 + 9, 64), 4), ((2, 256 * 70 + 9, 64), 19), ((2, 512 * 66, 64), 6), ((2, 512 * 300 + 1, 64), 41)])
def test_lost_summary_of_two_levels(gpu, shape, drop):
    torch, hb = gpu
    B, n, D = shape
    steps = hb.heinsen_tile_shape(B, D, n, hb.HEINSEN_LAYOUT_BND, 0)[1]
    rng = np.random.default_rng(n)
    a, b, x0 = cross._inputs(rng, shape, "BND", "signed")
    stream = torch.cuda.current_stream()
    want = cross._run(gpu, a, b, x0, "BND", (), False)
    assert hb.heinsen_check(stream) == hb.HEINSEN_OK
    try:
        hb.heinsen_test_carry(2000, drop, 0, stream)  # a few milliseconds of polling, then give up
        print(f"[lost] {shape}: tile {drop} does not publish", flush=True)
        got = cross._run(gpu, a, b, x0, "BND", (), False)
    finally:
        hb.heinsen_test_carry(0, 0xFFFFFFFF, 0, stream)
    assert hb.heinsen_check(stream) == hb.HEINSEN_ERR_CARRY_LOST
    assert hb.heinsen_check(stream) == hb.HEINSEN_OK
    chunk, col = divmod(drop, B)  # a column is an item
    first = (chunk + 1) * steps
    assert np.array_equal(got[col, :first].view(np.uint32), want[col, :first].view(np.uint32))
    assert np.isnan(got[col, first:]).all()
    assert np.array_equal(got[1 - col].view(np.uint32), want[1 - col].view(np.uint32))
    again = cross._run(gpu, a, b, x0, "BND", (), False)
    assert np.array_equal(again.view(np.uint32), want.view(np.uint32))


# Two carry levels, eight waves and tall tiles: behind one a_t = +inf every step of its channel is infinite, in the waves of its
# tile, the tiles of its group and the groups behind, from x_0 = 0 and with a restart (a_t = 0) before it as well.  Each is in 32
# steps (a lane's) of its own, with 32 steps at least before the infinite one.
@pytest.mark.parametrize("mode", ["signed", "positive", "positive_logout", "log_logout"])
@pytest.mark.parametrize("shape,steps", [((1, 1537, 64), 256), ((1, 256 * 18 + 5, 70), 256), ((9, 3000, 8), 256), ((12, 4096, 64), 256), ((2, 256 * 67, 64), 256),
                                         ((1, 512 * 130 + 9, 48), 512), ((1, 512 * 259, 64), 512), ((8, 512 * 18 + 3, 64), 512), ((40, 3000, 64), 512)])
def test_behind_an_infinite_coefficient_all_is_infinite(gpu, mode, shape, steps):
    torch, hb = gpu
    B, n, D = shape
    assert hb.heinsen_tile_shape(B, D, n, hb.HEINSEN_LAYOUT_BND, hb.flags_from_names(cross.MODES[mode]))[1] == steps
    rng = np.random.default_rng(sum(shape))
    a, b = rng.uniform(0.4, 1.0, shape).astype(np.float32), rng.uniform(0.1, 1.0, shape).astype(np.float32)
    x0 = np.where(rng.random(B * D) < 0.5, 0.0, 1.0).astype(np.float32)
    at = rng.integers(32, n, (B, D))
    at[0, :8] = 32 + np.arange(8) * (steps // 8)  # every wave of the first tile
    restart = at // 32 * 32 - rng.integers(1, 2000, (B, D))
    t = np.arange(n)[None, :, None]
    a[t == restart[:, None]] = 0.0
    a[t == at[:, None]] = np.inf
    with np.errstate(divide="ignore"):
        stored = [np.log(v) for v in (a, b, x0)] if mode == "log_logout" else (a, b, x0)
    print(f"[to infinity] {mode} shape={shape}", flush=True)
    got = cross._run(gpu, *stored, "BND", cross.MODES[mode], False)
    assert np.array_equal(got == np.inf, np.broadcast_to(t >= at[:, None], shape)) and not np.isnan(got).any()


# The same by growth, without logarithms: products of a few waves leave float32, and are zero in the tiles before that.
@pytest.mark.parametrize("shape", [(1, 1537, 64), (1, 256 * 18 + 5, 70), (9, 3000, 8), (12, 4096, 64), (2, 256 * 67, 64)])
def test_growth_without_logarithms_ends_in_infinity(gpu, shape):
    B, n, D = shape
    x0 = np.ones(B * D, np.float32)
    t = np.arange(n)[None, :, None]
    for grow in (2.1, 3.0, 5.0):
        for begin in (0, 40, 300, 700, 1300):
            a = np.broadcast_to(np.where(t < begin, 0.5, grow), shape).astype(np.float32)
            b = np.full(shape, 0.5, np.float32)
            print(f"[growth] shape={shape} {grow} from {begin} on", flush=True)
            got = cross._run(gpu, a, b, x0, "BND", cross.MODES["linear"], False)
            with np.errstate(over="ignore"):
                ref = oracle.sequential(a, b, x0, layout=oracle.LAYOUT_BND)
            assert np.all(got[ref > 3.5e38] == np.inf)
            small = ref < 1e37
            assert np.all(np.abs(got[small] - ref[small]) <= 1e-5 * ref[small])


# Items of fewer than 32 channels, whose runs are dealt out through LDS: one wave's worth of steps more than the short
# kernels take, tiles that end in the middle of a wave and of a vector, runs that begin on any element (odd n * D), the
# last column with fewer items than the others, one item alone, one more item than a column, both numbers of items per
# column, groups of four and of eight tiles with one and two carry levels (whole runs and halves).
@pytest.mark.parametrize("mode", ["signed", "log_logout", "linear"])
@pytest.mark.parametrize("bf16", [False, True])
@pytest.mark.parametrize("shape", [
    (1, 129, 2), (33, 160, 2), (22, 257, 3), (17, 288, 4), (70, 511, 5), (1, 1024, 31), (3, 1025, 31), (5, 300, 16), (64, 255, 9),
    (800, 333, 9), (700, 300, 19), (200, 1100, 13), (3, 2049, 23), (25, 2304, 31), (19, 3001, 30), (2, 20001, 7), (40, 1055, 1 + 16),
])
def test_runs_of_narrow_items(gpu, mode, bf16, shape):
    rng = np.random.default_rng(sum(shape) + int(bf16))
    a, b, x0 = cross._inputs(rng, shape, "BND", mode)
    if bf16:  # the bf16-rounded values are what is stored: they define the problem
        a = workloads.bf16_bits_to_f32(workloads.f32_to_bf16_bits(a)).reshape(a.shape)
        b = workloads.bf16_bits_to_f32(workloads.f32_to_bf16_bits(b)).reshape(b.shape)
    for offset in (0, 1, 3):
        print(f"[runs] {mode} bf16={bf16} shape={shape} offset={offset}", flush=True)
        got = cross._run(gpu, a, b, x0, "BND", cross.MODES[mode], bf16, offset_elems=offset)
        cross._check(got, a, b, x0, "BND", mode)


# The last steps of a sequence, fewer than a wave takes, are loaded one by one and in bf16 widened afterwards: every number of
# them, in narrow items and wide rows, a wave each and several, identity elements of numbers (1, 0) and of logarithms (0, -inf).
@pytest.mark.parametrize("mode", ["signed", "log_logout", "linear"])
def test_last_steps_of_every_length_in_bf16(gpu, mode):
    rng = np.random.default_rng(7)
    for last in range(1, 32):
        for shape in [(3, 128 + 32 * (last % 4) + last, 7), (2, 8 + last, 96), (2, 64 + last, 40), (1, 256 * (last % 3) + last + 160, 130)]:
            a, b, x0 = cross._inputs(rng, shape, "BND", mode)
            a, b = (workloads.bf16_bits_to_f32(workloads.f32_to_bf16_bits(v)).reshape(v.shape) for v in (a, b))
            print(f"[last steps] {mode} shape={shape}", flush=True)
            cross._check(cross._run(gpu, a, b, x0, "BND", cross.MODES[mode], True), a, b, x0, "BND", mode)


# Output that a wave writes in whole lines goes through the L2 at once: rows of a multiple of 32 channels from an address
# that is one of 128 bytes (offsets 0 and 32; offset 1: any other), one wave to eight per tile, one tile and several,
# columns across items, wide tiles, single values and pairs.
@pytest.mark.parametrize("mode", ["signed", "log_logout", "signed_clog"])
@pytest.mark.parametrize("shape", [
    (2, 17, 32), (2, 40, 64), (3, 100, 96), (3, 300, 64), (1, 2500, 160), (2, 700, 1024), (9, 513, 32), (128, 1030, 256),
])
def test_output_written_through(gpu, mode, shape):
    rng = np.random.default_rng(sum(shape))
    a, b, x0 = cross._inputs(rng, shape, "BND", mode)
    for offset in (0, 32, 1):
        print(f"[through] {mode} shape={shape} offset={offset}", flush=True)
        got = cross._run(gpu, a, b, x0, "BND", cross.MODES[mode], False, offset_elems=offset)
        cross._check(got, a, b, x0, "BND", mode)


def test_fewer_records_where_the_fixed_scratch_is_short(gpu):
    """40 columns of 1000 tiles need 6.4e6 records with one carry level, 5.2e6 with two; the fixed array holds 6.29e6.
    The values are x_t = 1 for a = 1/2, b = 1/2, x_0 = 1."""
    torch, hb = gpu
    B, n, D = 40, 256 * 1000, 64
    a = torch.full((B, n, D), 0.5, dtype=torch.bfloat16, device="cuda")
    x0 = torch.ones(1, dtype=torch.float32, device="cuda")
    out = torch.empty((B, n, D), dtype=torch.float32, device="cuda")
    flags = hb.HEINSEN_IN_BF16 | hb.HEINSEN_X0_SCALAR
    for call in (hb.heinsen_scan_static, hb.heinsen_scan):
        out.fill_(float("nan"))
        call(a, a, x0, out, B, D, n, hb.HEINSEN_LAYOUT_BND, flags, torch.cuda.current_stream())
        assert hb.heinsen_check(torch.cuda.current_stream()) == hb.HEINSEN_OK
        assert float((out - 1.0).abs().max()) <= 1e-5


def test_a_tile_that_never_publishes_ends_in_nan_with_two_carry_levels(gpu):
    torch, hb = gpu
    B, n, D = 1, 256 * 100, 128  # two columns
    a = torch.full((B, n, D), 0.5, device="cuda")
    x0 = torch.ones(D, device="cuda")
    out = torch.empty((B, n, D), device="cuda")
    args = (a, a, x0, out, B, D, n, hb.HEINSEN_LAYOUT_BND, 0, torch.cuda.current_stream())
    hb.heinsen_scan(*args)
    torch.cuda.synchronize()
    drop = 2 * 10  # chunk 10 of column 0
    try:
        hb.heinsen_test_carry(spin_limit=200, drop_tile=drop)
        out.fill_(0.0)
        hb.heinsen_scan(*args)
        assert hb.heinsen_check(torch.cuda.current_stream()) == hb.HEINSEN_ERR_CARRY_LOST
    finally:
        hb.heinsen_test_carry()
    assert torch.isnan(out[0, 256 * 11:, :64]).all()
    assert (out[0, : 256 * 11, :64] - 1).abs().max() <= 1e-5 and (out[0, :, 64:] - 1).abs().max() <= 1e-5
    hb.heinsen_scan(*args)
    assert hb.heinsen_check(torch.cuda.current_stream()) == hb.HEINSEN_OK
    assert (out - 1).abs().max() <= 1e-5


# Calls large enough to go through the L2 (rows that do not keep to 128-byte lines) or past the caches with columns
# across items or narrow items as runs: one batch item against the oracle, the others bit for bit the same (a channel's arithmetic does not depend
# on where it lies).  More than 192 MiB of output; bf16 288 MiB, narrow items 192 MiB of input and output.
@pytest.mark.parametrize("mode,bf16,shape", [
    ("signed", False, (8, 5000, 1501)), ("log_logout", False, (12, 6000, 770)), ("signed", True, (16, 8192, 301)),
    ("log", True, (16, 8192, 301)), ("signed_clog", False, (20, 4500, 301)), ("signed_clog", True, (32, 4500, 200)),
    ("positive", False, (130, 6300, 65)), ("signed", False, (256, 4096, 19)), ("signed", True, (300, 4100, 30)),
    ("signed", False, (260, 2048, 96)), ("linear", False, (8, 5000, 1501)),
    # narrow items as runs: past the caches, on lines and not, whole runs and halves (two carry levels), and with ordinary stores
    ("signed", False, (700, 4099, 19)), ("log_logout", True, (700, 4099, 19)), ("linear", False, (512, 6400, 16)),
    ("signed", False, (2, 2000003, 13)), ("signed", True, (2, 2000003, 13)), ("signed", False, (544, 1294, 19)),
    # wide tiles whose items lie a power of two apart
    ("signed", False, (16, 1024, 2048)), ("signed", True, (16, 2048, 2048)),
])
def test_large_calls_item_by_item(gpu, mode, bf16, shape):
    torch, hb = gpu
    B, n, D = shape
    print(f"[large] {mode} bf16={bf16} shape={shape}", flush=True)
    rng = np.random.default_rng(B * D + int(bf16))
    a, b, x0 = cross._inputs(rng, (1, n, D), "BND", mode)
    if bf16:
        a = workloads.bf16_bits_to_f32(workloads.f32_to_bf16_bits(a)).reshape(a.shape)
        b = workloads.bf16_bits_to_f32(workloads.f32_to_bf16_bits(b)).reshape(b.shape)
    kind = torch.bfloat16 if bf16 else torch.float32
    ta, tb = (torch.from_numpy(v).cuda().to(kind).expand(B, n, D).contiguous() for v in (a, b))
    tx = torch.from_numpy(x0).cuda().repeat(B)
    out = torch.full((B, n, D) + ((2,) if mode == "signed_clog" else ()), float("nan"), device="cuda")
    flags = hb.flags_from_names(cross.MODES[mode]) | (hb.HEINSEN_IN_BF16 if bf16 else 0)
    hb.heinsen_scan(ta, tb, tx, out, B, D, n, hb.HEINSEN_LAYOUT_BND, flags, torch.cuda.current_stream())
    torch.cuda.synchronize()
    first = out[:1]
    assert all(torch.equal(out[i].view(torch.int32), first[0].view(torch.int32)) for i in range(1, B))
    cross._check(first.cpu().numpy(), a, b, x0, "BND", mode)


# Slow decay (a within 1e-4 of one, x close to 1), log domain throughout: the error of the states that travel between
# tiles, since the steps inside a tile add little.  A fold of eight tile summaries in float32 rounds a term of size 1 to
# 2^-24 (6e-8) up to eight times over; in float64 what is left is the outputs' own rounding and that of one tile.
# Measured relative rms over the steps behind the first super-group, 4 and 12 columns: 1.0e-7 and 1.1e-7 with the
# levels above a tile in float64, 1.5e-7 with them in float32.
@pytest.mark.parametrize("columns", [4, 12])
def test_summaries_of_many_tiles_keep_float64(gpu, columns):
    rng = np.random.default_rng(1)
    shape = (1, 256 * 150 + 17, 64 * columns)
    a = np.exp(-1e-4 * rng.uniform(0.5, 1.5, shape)).astype(np.float32)
    b = ((1 - a.astype(np.float64)) * rng.uniform(0.9, 1.1, shape)).astype(np.float32)
    a, b, x0 = np.log(a), np.log(b), np.zeros(shape[2], np.float32)
    got = cross._run(gpu, a, b, x0, "BND", cross.MODES["log_logout"], False)
    behind = slice(256 * 64, None)
    err = got[:, behind].astype(np.float64) - oracle.sequential_log(a, b, x0, layout=oracle.LAYOUT_BND)[:, behind]
    rms = float(np.sqrt(np.mean(err * err)))  # of log x, which is the relative error of x
    assert rms <= 1.25e-7, rms


# The same where eight waves keep the sequence in 84 tiles, and in tall tiles, with 44 of them behind the first super-group.
@pytest.mark.parametrize("shape,steps", [((1, 256 * 84, 192), 256), ((1, 512 * 300 + 17, 64), 512), ((2, 512 * 300 + 17, 64), 512)])
def test_states_behind_a_super_group_keep_float64(gpu, shape, steps):
    torch, hb = gpu
    B, n, D = shape
    flags = hb.flags_from_names(cross.MODES["log_logout"])
    assert hb.heinsen_tile_shape(B, D, n, hb.HEINSEN_LAYOUT_BND, flags)[1] == steps
    rng = np.random.default_rng(1)
    a = np.exp(-1e-4 * rng.uniform(0.5, 1.5, shape)).astype(np.float32)
    b = ((1 - a.astype(np.float64)) * rng.uniform(0.9, 1.1, shape)).astype(np.float32)
    a, b, x0 = np.log(a), np.log(b), np.zeros(B * D, np.float32)
    print(f"[float64] shape={shape}", flush=True)
    got = cross._run(gpu, a, b, x0, "BND", cross.MODES["log_logout"], False)
    behind = slice(64 * 256 if steps == 256 else 256 * 512, None)
    err = got[:, behind].astype(np.float64) - oracle.sequential_log(a, b, x0, layout=oracle.LAYOUT_BND)[:, behind]
    rms = float(np.sqrt(np.mean(err * err)))
    print(f"[float64] shape={shape} rms {rms:.3g}", flush=True)
    assert rms <= 1.25e-7, rms


# Tall tiles, the second half of a tile: logarithms, no input.  Of every three tiles the first adds a small number e to log x, the second
# takes a large one off and the third adds the large one again in its first half, in the same float32.  What its second half starts
# from is the sum of the e.  Formed in float32, from a state at its start of about -1000, it would have few bits of e (2^-14 in the
# base-2 logarithm, 4e-5).  Bound: e is rounded when it is converted to base 2, by at most 0.1 * 2^-23 each of up to 100
# times (1.2e-6), and the sum, below 4, three times on its way out (7e-7).
@pytest.mark.parametrize("shape", [(1, 512 * 300 + 17, 64), (8, 512 * 18, 64), (40, 512 * 45 + 3, 5)])
def test_second_halves_of_tall_tiles_start_from_float64(gpu, shape):
    torch, hb = gpu
    B, n, D = shape
    flags = hb.flags_from_names(cross.MODES["log_logout"])
    assert hb.heinsen_tile_shape(B, D, n, hb.HEINSEN_LAYOUT_BND, flags)[1] == 512
    rng = np.random.default_rng(n)
    times = n // 1536
    e, large = rng.uniform(-0.1, 0.1, (B, times, D)).astype(np.float32), rng.uniform(900, 1000, (B, times, D)).astype(np.float32)
    a, b, x0 = np.zeros(shape, np.float32), np.full(shape, -np.inf, np.float32), np.zeros(B * D, np.float32)
    at = np.arange(times)[None, :, None] * 1536 + rng.integers(0, 256, (3, B, times, D))
    i, j = np.arange(B)[:, None, None], np.arange(D)[None, None, :]
    a[i, at[0], j] = e
    a[i, at[1] + 512, j] = -large
    a[i, at[2] + 1024, j] = large
    print(f"[halves] shape={shape}", flush=True)
    got = cross._run(gpu, a, b, x0, "BND", cross.MODES["log_logout"], False)
    last = got[:, :times * 1536].reshape(B, times, 1536, D)[:, :, 1280:].astype(np.float64)  # the second halves of the third tiles
    want = np.cumsum(e.astype(np.float64), axis=1)[:, :, None]
    assert np.abs(want).max() < 4
    assert np.abs(last - want).max() <= 2e-6


# a few steps: four channels per thread and one, the ends of a workgroup, the last length of the kernel and the next
@pytest.mark.parametrize("mode", ["signed", "positive"])
@pytest.mark.parametrize("bf16", [False, True])
def test_a_few_steps(gpu, mode, bf16):
    rng = np.random.default_rng(91 + int(bf16))
    for shape in [(1, 1, 2), (2, 1, 4), (64, 1, 1024), (3, 2, 341), (5, 3, 205), (1, 7, 1028), (2, 8, 260), (7, 8, 37), (2, 9, 260)]:
        a, b, x0 = cross._inputs(rng, shape, "BND", mode)
        if bf16:  # the bf16-rounded values are what is stored: they define the problem
            a = workloads.bf16_bits_to_f32(workloads.f32_to_bf16_bits(a)).reshape(a.shape)
            b = workloads.bf16_bits_to_f32(workloads.f32_to_bf16_bits(b)).reshape(b.shape)
        for offset in (0, 1, 4):
            print(f"[steps] {mode} bf16={bf16} shape={shape} offset={offset}", flush=True)
            got = cross._run(gpu, a, b, x0, "BND", cross.MODES[mode], bf16, offset_elems=offset)
            cross._check(got, a, b, x0, "BND", mode)


def test_a_few_steps_out_of_range_and_back(gpu):
    """States beyond float32 between outputs, zeros, infinities and NaN: as the definition has them."""
    # all factors and float32 outputs are normal numbers (at least 2^-126 = 1.18e-38) except x_0 = 1e-39, which counts as 0
    a = np.tile(np.array([1e30, 1e30, 1e-30, 1e-37], np.float32)[None, :, None], (1, 1, 8))
    b = np.zeros_like(a)
    x0 = np.array([1.0, -1.0, 0.0, np.inf, np.nan, 1e-30, 1e-39, 2.0], np.float32)
    a[0, 1, 7], b[0, 1, 7] = 0.0, 3.0
    got = cross._run(gpu, a, b, x0, "BND", (), False)[0]
    inf = np.inf
    want = np.array([[1e30, -1e30, 0, inf, np.nan, 1.0, 0, 2e30], [inf, -inf, 0, inf, np.nan, 1e30, 0, 3.0],
                     [1e30, -1e30, 0, inf, np.nan, 1.0, 0, 3e-30], [1e-7, -1e-7, 0, inf, np.nan, 1e-37, 0, 0]])
    assert np.allclose(got, want, rtol=1e-6, atol=0, equal_nan=True)
