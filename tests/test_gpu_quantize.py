"""GPU parity: adapt_quantize / adapt_quantize_batched against the CPU oracle, bit for bit
(Sec. 3.2 SR rule; Alg. 1 per-layer Quantize)."""
import numpy as np
import pytest
import torch

import paper_2107_13490_amd as pkg
import workloads as wk
from oracle import fxp_oracle as orc

from gpu_util import ctx, dev, host, u64

pytestmark = pytest.mark.gpu


def _check(x, wl, fl, mode, seed, stream):
    q, cnt = ctx().quantize(dev(x), wl, fl, mode, seed, stream)
    want, nnz, sat = orc.quantize(x, wl, fl, mode, seed, stream)
    got = host(q)
    assert got.dtype == (np.int8 if wl <= 8 else np.int16)
    assert np.array_equal(got.astype(np.int64), want)
    assert u64(cnt).tolist() == [nnz, sat]


@pytest.mark.parametrize("n", [1, 7, 8, 9, 63, 1000, 2048 * 8 + 5, (1 << 20) + 3])
@pytest.mark.parametrize("wl,fl", [(8, 5), (12, 9), (4, 1), (16, 13), (2, 0)])
def test_sizes_and_formats(n, wl, fl):
    x = (np.random.default_rng(n + wl).standard_normal(n) * 2.0 ** (wl - 2 - fl)).astype(np.float32)
    _check(x, wl, fl, pkg.SR, seed=3, stream=n)


@pytest.mark.parametrize("wl,fl", [(8, 4), (16, 8), (8, 12), (3, 31), (16, 0)])
@pytest.mark.parametrize("mode", [pkg.SR, pkg.RN_HALF_UP])
def test_modes_seeds_streams(wl, fl, mode):
    x = (np.random.default_rng(7).standard_normal(40001) * 2.0 ** (wl - 1 - fl) * 0.6).astype(np.float32)
    _check(x, wl, fl, mode, seed=(5 << 40) + 17, stream=(9 << 35) + 2)
    _check(x, wl, fl, mode, seed=0, stream=0)


def test_special_values_and_denormals():
    den = np.float32(1e-45)
    base = np.array([np.nan, np.inf, -np.inf, -0.0, 0.0, den, -den, 3.4e38, -3.4e38, 1e-39, -1e-39,
                     7.9999, -8.0, -8.0001, 0.03125, -0.03125], dtype=np.float32)
    x = np.tile(base, 37)[:-3]
    for wl, fl in ((8, 4), (16, 12)):
        for seed in range(4):
            _check(x, wl, fl, pkg.SR, seed, 1)
        _check(x, wl, fl, pkg.RN_HALF_UP, 0, 0)


def test_grid_points_unchanged_for_any_seed():
    codes = np.arange(-128, 128).repeat(9)
    x = (codes * 2.0 ** -5).astype(np.float32)
    for seed in range(3):
        q, _ = ctx().quantize(dev(x), 8, 5, pkg.SR, seed, 4)
        assert np.array_equal(host(q).astype(np.int64), codes)


def test_empty_tensor():
    x = torch.empty(0, dtype=torch.float32, device="cuda")
    q, cnt = ctx().quantize(x, 8, 4)
    assert u64(cnt).tolist() == [0, 0] and q.numel() == 0


def test_config2_full_size_tensors():
    L = wk.config2()
    for stream, t in enumerate((L.x, L.w, L.dy)):
        _check(t.ravel(), L.wl, L.fl, pkg.SR, seed=0, stream=stream + 1)


def test_config3_weights_keep_exact_zeros():
    L = wk.config3(batch=2)
    q, cnt = ctx().quantize(dev(L.w.ravel()), L.wl, L.fl, pkg.SR, 0, 2)
    got = host(q)
    assert (got[L.w.ravel() == 0] == 0).all()
    want, nnz, sat = orc.quantize(L.w.ravel(), L.wl, L.fl, pkg.SR, 0, 2)
    assert np.array_equal(got.astype(np.int64), want) and u64(cnt).tolist() == [nnz, sat]


def test_batched_matches_oracle():
    g = np.random.default_rng(1)
    sizes = [1, 5, 4096, 100003, 0, 17, 300000, 8]
    fmts = [(8, 4), (12, 9), (4, 2), (16, 10), (8, 4), (6, 3), (8, 5), (9, 4)]
    xs = [(g.standard_normal(n) * 2.0 ** (f[0] - 2 - f[1])).astype(np.float32) for n, f in zip(sizes, fmts)]
    streams = list(range(10, 10 + len(xs)))
    outs, cnt = ctx().quantize_batched([dev(x) for x in xs], fmts, streams, pkg.SR, seed=77)
    c = u64(cnt)
    for t, (x, f) in enumerate(zip(xs, fmts)):
        want, nnz, sat = orc.quantize(x, f[0], f[1], pkg.SR, 77, streams[t])
        assert np.array_equal(host(outs[t]).astype(np.int64), want)
        assert c[2 * t:2 * t + 2].tolist() == [nnz, sat]


def test_batched_many_items():
    g = np.random.default_rng(2)
    xs = [(g.standard_normal(100 + 37 * t)).astype(np.float32) for t in range(150)]
    fmts = [(8, 4) if t % 2 else (12, 8) for t in range(150)]
    outs, cnt = ctx().quantize_batched([dev(x) for x in xs], fmts, list(range(150)), pkg.SR, seed=1)
    c = u64(cnt)
    for t in (0, 1, 63, 64, 65, 127, 128, 149):
        want, nnz, sat = orc.quantize(xs[t], fmts[t][0], fmts[t][1], pkg.SR, 1, t)
        assert np.array_equal(host(outs[t]).astype(np.int64), want)
        assert c[2 * t:2 * t + 2].tolist() == [nnz, sat]


# around the largest call whose counters are summed by the launch itself (192 chunks of 2048 elements on at most 64
# blocks; 4 tensors of together 128 chunks), each twice, so that a ticket left behind would show
@pytest.mark.parametrize("n", [2048, 64 * 2048 + 1, 128 * 2048 + 8, 192 * 2048, 192 * 2048 + 1, 255 * 2048 + 9, 256 * 2048, 256 * 2048 + 1])
@pytest.mark.parametrize("wl", [8, 12])
def test_counters_of_single_and_two_launch_sizes(n, wl):
    x = np.random.default_rng(n).standard_normal(n).astype(np.float32)
    for _ in range(2):
        _check(x, wl, wl - 2, pkg.SR, seed=3, stream=n)


@pytest.mark.parametrize("sizes", [[3000] * 15, [3000] * 16, [3000] * 17, [100 * 2048, 156 * 2048], [100 * 2048, 156 * 2048 + 1], [0, 5],
                                   [3000] * 4, [3000] * 5, [70 * 2048 + 3, 0, 9, 56 * 2048], [64 * 2048, 64 * 2048], [64 * 2048 + 1, 64 * 2048]])
def test_batched_counters_of_single_and_two_launch_calls(sizes):
    g = np.random.default_rng(sum(sizes) + len(sizes))
    xs = [g.standard_normal(n).astype(np.float32) for n in sizes]
    fmts = [(8, 6) if t % 2 else (12, 10) for t in range(len(sizes))]
    for _ in range(2):
        _, cnt = ctx().quantize_batched([dev(x) for x in xs], fmts, list(range(len(xs))), pkg.SR, seed=5)
        want = [c for t, x in enumerate(xs) for c in orc.quantize(x, fmts[t][0], fmts[t][1], pkg.SR, 5, t)[1:]]
        assert u64(cnt)[:len(want)].tolist() == want


def test_invalid_arguments_are_rejected():
    x = torch.zeros(64, dtype=torch.float32, device="cuda")
    with pytest.raises(pkg.AdaptError) as e:
        ctx().quantize(x, 33, 4)
    assert e.value.status == -1
    with pytest.raises(pkg.AdaptError):
        ctx().quantize(x, 8, 32)
    with pytest.raises(pkg.AdaptError):
        ctx().quantize(x[1:], 8, 4)          # misaligned
    with pytest.raises(pkg.AdaptError):
        ctx().quantize(x, 8, 4, mode=5)


def test_batched_ranges_feed_the_precision_search():
    rng = np.random.default_rng(21)
    xs = [(rng.standard_normal(n) * sc).astype(np.float32) for n, sc in ((110592, 0.06), (7, 3.0), (40000, 1e-3), (1, 1.0))]
    xs[0][[5, 77, 1000]] = [np.inf, -np.inf, np.nan]          # non-finite values are left out of the range
    xs.append(np.full(16, np.nan, dtype=np.float32))           # no finite element: (+inf, -inf)
    fmts = [(8, 5), (12, 9), (8, 7), (4, 1), (8, 5)]
    ranges = torch.empty(2 * len(xs), dtype=torch.float32, device="cuda")
    outs, cnt = ctx().quantize_batched([dev(x) for x in xs], fmts, list(range(1, 6)), pkg.SR, 3, ranges=ranges)
    got = host(ranges).reshape(-1, 2)
    for t, x in enumerate(xs):
        want, nnz, sat = orc.quantize(x, fmts[t][0], fmts[t][1], orc.SR, 3, t + 1)
        assert np.array_equal(host(outs[t]).astype(np.int64), want)
        assert u64(cnt)[2 * t:2 * t + 2].tolist() == [nnz, sat]
        fin = x[np.isfinite(x)]
        if fin.size:
            assert (got[t, 0], got[t, 1]) == (fin.min(), fin.max())
        else:
            assert got[t, 0] == np.inf and got[t, 1] == -np.inf
    # the pair of the first tensor drives the search without a range pass
    res = ctx().kld_precision_search_ranged(dev(xs[0]), ranges[0:2], 4, 16, 3, 2048, 1e-2, stream=2)
    ref = orc.kld_precision_search(xs[0], 4, 16, 3, 2048, 1e-2, None, orc.SR, 0, 2)
    assert host(res["sel"]).tolist() == [ref["wl_sel"], ref["fl_sel"]]
    assert np.allclose(host(res["kld"]), ref["kld"], rtol=1e-5, atol=1e-12)
    # a mask: only tensor 2 is tracked, the others report (+inf, -inf)
    ctx().quantize_batched([dev(x) for x in xs], fmts, list(range(1, 6)), pkg.SR, 3, ranges=ranges, range_of=[2])
    got = host(ranges).reshape(-1, 2)
    assert (got[2, 0], got[2, 1]) == (xs[2].min(), xs[2].max())
    assert all(got[t, 0] == np.inf and got[t, 1] == -np.inf for t in (0, 1, 3, 4))
    # ranges without counters
    r2 = torch.empty(2, dtype=torch.float32, device="cuda")
    it = (pkg.binding.QuantizeItem * 1)(pkg.binding.QuantizeItem(dev(xs[2]).data_ptr(), outs[2].data_ptr(), xs[2].size, 8, 7, 3))
    assert pkg.load_library().adapt_quantize_batched_ranges(ctx().handle, it, 1, pkg.SR, 3, None, r2.data_ptr(), 1) == 0
    assert host(r2).tolist() == [float(xs[2].min()), float(xs[2].max())]


@pytest.mark.parametrize("wl,n", [(8, 270_000_003), (12, 135_000_005)])
@pytest.mark.parametrize("batched", [False, True])
def test_codes_that_exceed_the_last_level_cache(wl, n, batched):
    # codes of more than 256 MB take other stores; slices at both ends and inside against the oracle, the counters against the codes
    x = torch.randn(n, device="cuda")
    if batched:
        (q,), counters = ctx().quantize_batched([x], [(wl, wl - 3)], [9], pkg.SR, 5)[:2]
        counters = u64(counters).ravel()
    else:
        q, counters = ctx().quantize(x, wl, wl - 3, pkg.SR, 5, 9)
        counters = u64(counters)
    for a in (0, 8 * 262144 - 50, n // 2 + 3, n - 3000):
        part = host(x[a:a + 3000])
        bits = orc.r16(5, 9, np.arange(a, a + part.size, dtype=np.uint64))
        want = orc.quantize_with_bits(part, wl, wl - 3, bits)[0]
        assert np.array_equal(host(q[a:a + 3000]).astype(np.int64), want), a
    assert int(counters[0]) == int(torch.count_nonzero(q))
