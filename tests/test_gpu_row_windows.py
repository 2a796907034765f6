"""Rows of [B, D, n] that begin and end anywhere relative to the 16-byte boundaries: every length around the
edges of a vector, a lane, a wave and a workgroup, pointers that start off a boundary together, few rows and
many (the plan changes at 512), and the ranges in which a complex output is evaluated in float64."""
import numpy as np
import pytest

import oracle
from paper_2311_06281_amd import workloads

import test_gpu_cross_product as cross
from test_gpu_cross_product import gpu  # noqa: F401  (fixture)

pytestmark = pytest.mark.gpu

# (rows, n): one and several rows per wave, ends of lanes of 8, 16 and 32 steps, of waves and of tiles
SHAPES = [(5, 1), (300, 2), (131, 3), (700, 7), (65, 9), (130, 13), (77, 31), (64, 33), (40, 63), (33, 101), (20, 129), (21, 249),
          (9, 255), (600, 257), (3, 300), (530, 389), (520, 505), (515, 511), (6, 513), (70, 1017), (66, 1021), (65, 1025),
          (65, 2041), (64, 2045), (3, 2047), (513, 2047), (514, 2500), (2, 4093), (513, 3001), (2, 8191), (514, 4097),
          (2, 16382), (1, 16383), (1, 16385), (2, 24577)]


@pytest.mark.parametrize("mode", list(cross.MODES))
@pytest.mark.parametrize("bf16", [False, True])
def test_rows_off_the_vector_boundaries(gpu, mode, bf16):
    rng = np.random.default_rng(sum(map(ord, mode)) + int(bf16))
    for i, (rows, n) in enumerate(SHAPES):
        a, b, x0 = cross._inputs(rng, (1, rows, n), "BDN", mode)
        if bf16:  # the bf16-rounded values are what is stored: they define the problem
            a = workloads.bf16_bits_to_f32(workloads.f32_to_bf16_bits(a)).reshape(a.shape)
            b = workloads.bf16_bits_to_f32(workloads.f32_to_bf16_bits(b)).reshape(b.shape)
        for offset in ((0, 3) if i % 2 else (0, 4)):
            print(f"[windows] {mode} bf16={bf16} rows={rows} n={n} offset={offset}", flush=True)
            got = cross._run(gpu, a, b, x0, "BDN", cross.MODES[mode], bf16, offset_elems=offset)
            cross._check(got, a, b, x0, "BDN", mode)


# Positive numbers, so that nothing cancels and log x_t is as good as its largest term: every step of the
# log-domain form rounds a logarithm of size at most L to L 2^-24 (base 2), and n such roundings of
# random sign, five standard deviations of them, stay below 5 sqrt(n) L 2^-24 ln 2; 2e-6 for the
# hardware logarithm and exponential.  The float64 form rounds once.
@pytest.mark.parametrize("rows,n", [(60, 41), (20, 700), (12, 3001), (520, 1100)])
def test_complex_output_in_and_out_of_the_float64_range(gpu, rows, n):
    rng = np.random.default_rng(n)
    a = rng.uniform(0.7, 1.3, (rows, n)).astype(np.float32)
    b = rng.uniform(0.1, 1.0, (rows, n)).astype(np.float32)
    x0 = rng.uniform(0.5, 2.0, rows).astype(np.float32)
    at = n // 2
    a[0, at] = 1e-12           # below 2^-36
    a[1, at] = 1e6             # above 2^16
    a[2, at] = 0.0             # restarts the row
    b[3, at] = 1e-25           # below 2^-60
    b[4, at] = 1e25            # above 2^60
    b[5] = 0.0                 # only x_0
    x0[6] = 0.0
    x0[7], b[7] = 0.0, 0.0     # x = 0 throughout
    a[8], b[8] = 3.0, 0.0      # leaves float64 where n is long enough
    a[9], b[9] = 2.0 ** -7, 0.0
    a[10], b[10] = 2.0 ** -36, 1.0
    a[11, : at], a[11, at:], b[11] = 2.0 ** -9, 2.0 ** 7, 0.0
    got = cross._run(gpu, a[None], b[None], x0, "BDN", cross.MODES["signed_clog"], False)[0]
    for r in list(range(12)) + [rows - 1]:
        # (the oracle's states leave float64 below 2^-1074: rows that only scale x_0 have a closed form)
        if np.all(b[r] == 0.0):
            with np.errstate(divide="ignore"):
                ref = np.log(np.abs(np.float64(x0[r]))) + np.cumsum(np.log(a[r].astype(np.float64))) + 0j
        else:
            ref = oracle.seq_clog_scaled(a[r], b[r], x0[r])
        re = got[r, :, 0].astype(np.float64)
        zero = np.isneginf(ref.real)
        assert np.array_equal(np.isneginf(re), zero), r
        assert np.all(got[r, ~zero, 1] == 0.0), r
        size = max(1.0, float(np.max(np.abs(ref.real[~zero]), initial=0.0)) / np.log(2.0))
        err = np.max(np.abs(re[~zero] - ref.real[~zero]), initial=0.0)
        assert err <= 5 * np.sqrt(n) * size * 2.0 ** -24 * np.log(2.0) + 2e-6, (r, err)


# A row's result is its own: with and without neighbours that need the log-domain steps, bit for bit.  Several rows per
# wave, with the ends of rows inside a vector (41, 7, 301), on vectors (40, 300) and many rows that share one (1, 2).
@pytest.mark.parametrize("bf16", [False, True])
@pytest.mark.parametrize("rows,n", [(130, 41), (130, 40), (200, 7), (700, 301), (700, 300), (600, 1), (600, 2), (90, 100)])
def test_complex_rows_do_not_depend_on_their_neighbours(gpu, rows, n, bf16):
    rng = np.random.default_rng(rows + n)
    a, b, x0 = cross._inputs(rng, (1, rows, n), "BDN", "signed_clog")
    a = np.where(np.abs(a) < 1e-3, np.float32(0.25), a)  # in range everywhere
    b = np.where(np.abs(b) < 1e-3, np.float32(0.25), b)
    if bf16:
        a = workloads.bf16_bits_to_f32(workloads.f32_to_bf16_bits(a)).reshape(a.shape)
        b = workloads.bf16_bits_to_f32(workloads.f32_to_bf16_bits(b)).reshape(b.shape)
    alone = cross._run(gpu, a, b, x0, "BDN", cross.MODES["signed_clog"], bf16)
    a2, b2, x2 = a.copy(), b.copy(), x0.copy()
    changed = np.arange(1, rows, 3)
    a2[0, changed, n // 2] = np.resize(np.array([2.0 ** 40, 2.0 ** -50, np.nan, np.inf], np.float32), len(changed))
    x2[changed[::5]] = 1e-38
    got = cross._run(gpu, a2, b2, x2, "BDN", cross.MODES["signed_clog"], bf16)
    kept = np.setdiff1d(np.arange(rows), changed)
    assert np.array_equal(got[0, kept].view(np.uint32), alone[0, kept].view(np.uint32))
    finite = changed[np.isfinite(a2[0, changed, n // 2])]
    cross._check(got[:, finite], a2[:, finite], b2[:, finite], x2[finite], "BDN", "signed_clog")


# In range, with resets and small coefficients in every row: the float64 path, in each of the three kernels.  What it
# rounds is the number to float32 (2^-25 of it), its mantissa's logarithm (2^-24) and the sum with the exponent
# (2^-24 of log2 x, of the result): 2^-23 (1 + |re|) leaves a factor of two.  Log-domain steps round a logarithm per step:
# 3e-7 to 6e-7 on these rows.
@pytest.mark.parametrize("bf16", [False, True])
@pytest.mark.parametrize("rows,n", [(600, 300), (600, 257), (520, 700), (520, 1001), (520, 3001), (12, 5000)])
def test_complex_output_in_range_is_evaluated_in_float64(gpu, rows, n, bf16):
    rng = np.random.default_rng(rows * n)
    a = rng.uniform(0.7, 1.3, (rows, n)).astype(np.float32)
    b = rng.uniform(0.1, 1.0, (rows, n)).astype(np.float32)
    x0 = rng.uniform(0.5, 2.0, rows).astype(np.float32)
    a[:, n // 3], a[:, n // 5], a[::2, n // 4] = 0.0, 2.0 ** -36, 2.0 ** 16
    if bf16:
        a = workloads.bf16_bits_to_f32(workloads.f32_to_bf16_bits(a)).reshape(a.shape)
        b = workloads.bf16_bits_to_f32(workloads.f32_to_bf16_bits(b)).reshape(b.shape)
    got = cross._run(gpu, a[None], b[None], x0, "BDN", cross.MODES["signed_clog"], bf16)[0]
    ref = np.log(oracle.sequential(a[None], b[None], x0, layout=oracle.LAYOUT_BDN)[0])
    assert np.all(got[..., 1] == 0.0)
    err = np.abs(got[..., 0] - ref) / (1.0 + np.abs(ref))
    print(f"[float64] {rows} x {n} bf16={bf16}: {err.max():.2e}", flush=True)
    assert err.max() <= 2.0 ** -23


# Complex rows on nine to 16 waves (up to 1024 threads and 147 KB of LDS): 512 rows of four kinds, the last of which leaves
# the float64 range at one step.  Bounds as above.
@pytest.mark.parametrize("bf16", [False, True])
@pytest.mark.parametrize("n,offset", [(8193, 0), (12000, 0), (12000, 1), (16381, 1), (16384, 0)])
def test_complex_rows_on_up_to_sixteen_waves(gpu, n, offset, bf16):
    torch, hb = gpu
    rng = np.random.default_rng(n + offset)
    rows = 512
    a = rng.uniform(0.7, 1.3, (4, n)).astype(np.float32)
    b = rng.uniform(0.1, 1.0, (4, n)).astype(np.float32)
    x0 = rng.uniform(0.5, 2.0, 4).astype(np.float32)
    a[:3, n // 3], a[3, n // 2] = 0.0, 2.0 ** 20
    if bf16:
        a = workloads.bf16_bits_to_f32(workloads.f32_to_bf16_bits(a)).reshape(a.shape)
        b = workloads.bf16_bits_to_f32(workloads.f32_to_bf16_bits(b)).reshape(b.shape)
    kind = torch.bfloat16 if bf16 else torch.float32

    def device(v):
        buf = torch.zeros(rows * n + 8, dtype=kind, device="cuda")
        buf[offset:offset + rows * n] = torch.from_numpy(v).cuda().to(kind).repeat(rows // 4, 1).reshape(-1)
        return buf, buf[offset:]

    keep_a, ta = device(a)
    keep_b, tb = device(b)
    tx = torch.from_numpy(x0).cuda().repeat(rows // 4)
    keep = torch.full((2 * (rows * n + 8),), float("nan"), device="cuda")
    out = keep[2 * offset:2 * (offset + rows * n)]
    print(f"[waves] n={n} offset={offset} bf16={bf16}", flush=True)
    hb.heinsen_scan(ta, tb, tx, out, 1, rows, n, hb.HEINSEN_LAYOUT_BDN, hb.flags_from_names(cross.MODES["signed_clog"]) |
                    (hb.HEINSEN_IN_BF16 if bf16 else 0), torch.cuda.current_stream())
    torch.cuda.synchronize()
    assert torch.isnan(keep[:2 * offset]).all() and torch.isnan(keep[2 * (offset + rows * n):]).all()
    ref = np.log(oracle.sequential(a[None], b[None], x0, layout=oracle.LAYOUT_BDN)[0])
    got = out.reshape(rows // 4, 4, n, 2)
    assert (got[..., 1] == 0).all()
    err = (got[..., 0].double() - torch.from_numpy(ref).cuda()).abs().amax(0).cpu().numpy()  # worst of the rows of a kind
    assert np.all(err[:3] <= 2.0 ** -23 * (1.0 + np.abs(ref[:3])))
    size = max(1.0, float(np.max(np.abs(ref[3]))) / np.log(2.0))
    assert np.max(err[3]) <= 5 * np.sqrt(n) * size * 2.0 ** -24 * np.log(2.0) + 2e-6


# Rows of one tile on all eight waves (8, 16 and 32 steps per lane; a last wave with few steps, with one, with none), of several
# half tiles, and so many rows that the tiles are whole ones: every wave begins with what the waves before it add up to.
@pytest.mark.parametrize("mode", ["signed", "log_logout", "positive", "signed_clog"])
@pytest.mark.parametrize("rows,n", [(2, 4096), (3, 3585), (1, 3583), (2, 8192), (1, 7169), (2, 16384), (1, 14337), (513, 12289), (2, 8192 * 2 + 1), (1, 8192 * 35), (140, 16400)])
def test_sums_of_the_waves_of_a_tile(gpu, mode, rows, n):
    rng = np.random.default_rng(rows + n)
    a, b, x0 = cross._inputs(rng, (1, rows, n), "BDN", mode)
    print(f"[waves] {mode} rows={rows} n={n}", flush=True)
    got = cross._run(gpu, a, b, x0, "BDN", cross.MODES[mode], False, offset_elems=0)
    cross._check(got, a, b, x0, "BDN", mode)


# A wave whose sum of logarithms is +inf (its last a_t is), or whose product leaves float32 where that of half of its steps does
# not: everything behind it is infinite, in the waves of its tile, which start from sums of waves, and in the tiles behind that one.
# (Rows begin on 16 bytes, so that tiles do too.)
@pytest.mark.parametrize("rows,n", [(2, 4096), (3, 3588), (2, 8192), (2, 16384), (1, 14337), (513, 14340), (2, 8192 * 2 + 4), (1, 8192 * 35), (140, 16400)])
def test_behind_a_wave_that_leaves_float32_all_is_infinite(gpu, rows, n):
    torch, hb = gpu
    for mode in ("linear", "positive", "positive_logout", "signed"):
        steps = hb.heinsen_tile_shape(1, rows, n, hb.HEINSEN_LAYOUT_BDN, hb.flags_from_names(cross.MODES[mode]))[1]
        for wave in range(min(8, (n - 1) // (steps // 8))):
            first, behind = wave * steps // 8, (wave + 1) * steps // 8
            a, b = np.full((1, rows, n), 1.0 if mode == "linear" else 0.5, np.float32), np.full((1, rows, n), 0.5, np.float32)
            if mode == "linear":
                a[:, :, first:behind] = 2.0 ** (192 * 8 / steps)
            else:
                a[:, :, behind - 1] = np.inf
            print(f"[to infinity] {mode} rows={rows} n={n} wave={wave}", flush=True)
            got = cross._run(gpu, a, b, np.ones(rows, np.float32), "BDN", cross.MODES[mode], False)
            assert np.all(got[:, :, behind:] == np.inf) and np.isfinite(got[:, :, :first]).all()
