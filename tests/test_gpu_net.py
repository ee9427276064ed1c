"""GPU parity: the element-wise integer operations of a chained step and the chained step itself
(Alg. 1 for one batch: forward pass on quantized layers, backward pass, update, Quantize) against
the CPU oracle, bit for bit: codes, shifts, sums of squares, master weights, counters, ranges."""
import numpy as np
import pytest
import torch

import paper_2107_13490_amd as pkg
import workloads as wk
from oracle import conv_oracle as co
from oracle import fxp_oracle as orc
from oracle import net_oracle as no
from paper_2107_13490_amd import ConvDesc, LayerDesc

from gpu_util import ctx, dev, host

pytestmark = pytest.mark.gpu


def _dt(wl):
    return np.int8 if wl <= 8 else np.int16 if wl <= 16 else np.int32


def _sumsq(st):
    return (st.g_sumsq_hi << 64) + st.g_sumsq


def _codes(rng, shape, wl, zero_frac=0.0):
    lim = 1 << (wl - 1)
    a = rng.integers(-lim, lim, shape)
    if zero_frac:
        a[rng.random(shape) < zero_frac] = 0
    return a.astype(_dt(wl))


# ---- pooling --------------------------------------------------------------------------------------------

@pytest.mark.parametrize("shape", [(2, 4, 6, 16), (3, 8, 8, 64), (1, 2, 2, 3), (5, 6, 4, 24), (2, 32, 32, 64), (4, 2, 10, 7)])
@pytest.mark.parametrize("wl", [3, 8, 12])
def test_maxpool_forward(shape, wl):
    rng = np.random.default_rng(sum(shape) + wl)
    y = _codes(rng, shape, wl)
    got = host(ctx().maxpool2_fwd(dev(y), wl))
    assert np.array_equal(got.astype(np.int64), no.maxpool2(y))


@pytest.mark.parametrize("shape", [(2, 4, 6, 16), (3, 8, 8, 64), (1, 2, 2, 3), (5, 6, 4, 24), (2, 16, 16, 192), (4, 2, 10, 7)])
@pytest.mark.parametrize("wl", [2, 4, 8, 16])
@pytest.mark.parametrize("relu,pool", [(True, True), (False, True), (True, False)])
def test_relu_pool_backward(shape, wl, relu, pool):
    rng = np.random.default_rng(sum(shape) + 7 * wl + relu + 2 * pool)
    y = _codes(rng, shape, wl, zero_frac=0.3)            # low word lengths and zeros: many ties
    if relu:
        y = np.maximum(y, 0)
    n, h, w, c = shape
    da = _codes(rng, (n, h // 2, w // 2, c) if pool else shape, wl)
    got = host(ctx().relu_pool_bwd(dev(da), dev(y), wl, relu, pool))
    assert np.array_equal(got.astype(np.int64), no.relu_pool_bwd(da, y, relu, pool))


def test_pooling_rejects_odd_maps_and_empty_batch_is_a_no_op():
    y = dev(np.zeros((1, 3, 4, 16), np.int8))
    with pytest.raises(pkg.AdaptError):
        ctx().maxpool2_fwd(y, 8, out=dev(np.zeros((1, 1, 2, 16), np.int8)))
    e = torch.empty((0, 4, 4, 16), dtype=torch.int8, device="cuda")
    assert ctx().maxpool2_fwd(e, 8).shape == (0, 2, 2, 16)


# ---- fitting requantization -----------------------------------------------------------------------------

@pytest.mark.parametrize("n", [1, 5, 8, 9, 2048, 100003, (1 << 20) + 1])
@pytest.mark.parametrize("bits,wl,mag", [(32, 8, 20), (32, 4, 30), (32, 12, 9), (64, 16, 45), (64, 8, 33), (32, 16, 14), (64, 2, 50)])
def test_requantize_fit(n, bits, wl, mag):
    rng = np.random.default_rng(n + wl + mag)
    acc = np.rint(rng.standard_normal(n) * 2.0 ** (mag - 2)).astype(np.int64)
    acc = np.clip(acc, -(1 << (bits - 2)), 1 << (bits - 2))
    d = dev(acc.astype(np.int32 if bits == 32 else np.int64))
    for mode in (pkg.SR, pkg.RN_HALF_UP):
        q, sh, ss = ctx().requantize_fit(d, wl, mode=mode, seed=3, stream=n)
        want, wsh, wss = no.requantize_fit(acc, wl, mode, 3, n)
        assert int(sh.item()) == wsh
        assert np.array_equal(host(q).astype(np.int64), want)
        assert int(ss.item()) == wss


# more than one group of eight per thread in the launch that sums the squares (256 blocks of 1024) and in the one that
# does not (2048 blocks of 256), with a remainder; around the size from which the first has 1024 threads (256 x 160 groups);
# the largest magnitude in the last element
@pytest.mark.parametrize("n,sums", [(2100003, True), (4200003, False), (1023 * 8 + 1, False), (327680, True), (327681, True), (327691, True)])
def test_requantize_fit_several_groups_per_thread(n, sums):
    rng = np.random.default_rng(n)
    acc = rng.integers(-(1 << 25), 1 << 25, n)
    acc[-1] = -(1 << 28) - 1
    q, sh, ss = ctx().requantize_fit(dev(acc.astype(np.int32)), 8, seed=3, stream=n, want_sumsq=sums)
    want, wsh, wss = no.requantize_fit(acc, 8, pkg.SR, 3, n)
    assert int(sh.item()) == wsh and np.array_equal(host(q).astype(np.int64), want)
    assert not sums or int(ss.item()) == wss


def test_requantize_fit_degenerate_inputs():
    z = dev(np.zeros(100, np.int32))
    q, sh, ss = ctx().requantize_fit(z, 8)
    assert int(sh.item()) == 0 and int(ss.item()) == 0 and not host(q).any()
    small = dev(np.array([-128, 127, 5], np.int32))            # 128 needs 8 magnitude bits: shift 1
    q, sh, ss = ctx().requantize_fit(small, 8, mode=pkg.RN_HALF_UP)
    want, wsh, wss = no.requantize_fit(np.array([-128, 127, 5]), 8, orc.RN_HALF_UP)
    assert int(sh.item()) == wsh == 1 and host(q).tolist() == want.tolist() and int(ss.item()) == wss
    e = torch.empty(0, dtype=torch.int32, device="cuda")
    q, sh, ss = ctx().requantize_fit(e, 8)
    assert int(sh.item()) == 0 and int(ss.item()) == 0
    # the second call in a row starts its sum from zero again
    big = dev(np.full(4096, 1000, np.int32))
    _, _, s1 = ctx().requantize_fit(big, 8)
    _, _, s2 = ctx().requantize_fit(big, 8)
    assert int(s1.item()) == int(s2.item())


# ---- residual addition ----------------------------------------------------------------------------------

@pytest.mark.parametrize("n", [3, 8, 1000, 65537])
@pytest.mark.parametrize("fa,fb,fo", [((8, 5), (8, 5), (8, 5)), ((8, 3), (12, 9), (8, 4)), ((12, 9), (8, 3), (16, 12)),
                                      ((16, 12), (16, 6), (8, 2)), ((8, 5), (8, 7), (12, 9)), ((16, 14), (8, 0), (16, 10)),
                                      ((12, 4), (16, 12), (12, 6)), ((8, 6), (16, 8), (8, 6))])
def test_residual_add(n, fa, fb, fo):
    rng = np.random.default_rng(n + fa[1] + 3 * fb[1] + fo[0])
    a, b = _codes(rng, n, fa[0]), _codes(rng, n, fb[0])
    for relu in (False, True):
        got = host(ctx().residual_add(dev(a), fa, dev(b), fb, fo, seed=5, stream=n, relu=relu))
        want = no.residual_add(a, fa[1], b, fb[1], fo[0], fo[1], orc.SR, 5, n, relu)
        assert np.array_equal(got.astype(np.int64), want)


# ---- the chained step -----------------------------------------------------------------------------------

def _run_chain(layers, fmts, n, seed, lr=0.05, l1=1e-4, l2=1e-3, wl_max=16, context=None):
    rng = np.random.default_rng(seed)
    first = layers[0]
    x = rng.standard_normal((n, first.h, first.w, first.c)).astype(np.float32)
    ws = [(rng.standard_normal((L.k, L.r, L.s, L.c)) * (1.5 / np.sqrt(L.r * L.s * L.c))).astype(np.float32) for L in layers]
    descs = [LayerDesc(ConvDesc(n, L.h, L.w, L.c, L.k, L.r, L.s, L.stride, L.pad), int(L.relu), int(L.pool)) for L in layers]
    wdev = [dev(w.copy()) for w in ws]
    net = pkg.Net(context if context is not None else ctx(), descs, wdev, wl_max=wl_max)
    for l, (wl, fl) in enumerate(fmts):
        net.set_format(l, wl, fl)
    s0 = 1000 + seed
    net.quantize_weights(seed=seed, stream=s0)
    net.forward(dev(x), seed=seed, stream=s0)
    wq = no.quantize_weights(layers, fmts, ws, seed, s0)
    fwd = no.forward(layers, fmts, wq, x, seed, s0)
    last = len(layers) - 1
    assert np.array_equal(host(net.tensor(0, pkg.NT_INPUT)).astype(np.int64), fwd["a_in"].ravel())
    for l in range(len(layers)):
        assert np.array_equal(host(net.tensor(l, pkg.NT_QW)).astype(np.int64), wq[l].ravel()), l
        assert np.array_equal(host(net.tensor(l, pkg.NT_Y)).astype(np.int64), fwd["y"][l].ravel()), l
        assert np.array_equal(host(net.tensor(l, pkg.NT_A)).astype(np.int64), fwd["a"][l].ravel()), l
    # loss gradient: computed once on the host from the (identical) logits, handed to both sides
    wl_last, fl_last = fmts[last]
    logits = fwd["a"][last].reshape(n, -1) / 2.0 ** fl_last
    e = np.exp(logits - logits.max(axis=1, keepdims=True))
    soft = e / e.sum(axis=1, keepdims=True)
    soft[np.arange(n), rng.integers(0, soft.shape[1], n)] -= 1.0
    lim = 1 << (wl_last - 1)
    dl = np.clip(np.rint(soft * (lim - 1)), -lim, lim - 1).astype(_dt(wl_last))
    net.backward(dev(dl), 0, seed=seed, stream=s0)
    bwd = no.backward(layers, fmts, wq, fwd, dl, seed, s0)
    for l in range(len(layers)):
        st = net.tensor(l, pkg.NT_STATS)
        assert np.array_equal(host(net.tensor(l, pkg.NT_G)).astype(np.int64), bwd["g"][l].ravel()), l
        assert st.shift_w == bwd["shift_w"][l] and (_sumsq(st) if fmts[l][0] > 16 else st.g_sumsq) == bwd["sumsq"][l], l
        if layers[l].relu or layers[l].pool:
            assert np.array_equal(host(net.tensor(l, pkg.NT_DY)).astype(np.int64), bwd["dy"][l].ravel()), l
        if l > 0:
            assert st.shift_a == bwd["shift_a"][l], l
            assert np.array_equal(host(net.tensor(l - 1, pkg.NT_DA)).astype(np.int64), bwd["da"][l - 1].ravel()), l
    net.update(lr, l1, l2, seed=seed, stream=s0)
    upd = no.update(layers, fmts, ws, bwd, lr, l1, l2, seed, s0)
    for l in range(len(layers)):
        st = net.tensor(l, pkg.NT_STATS)
        assert np.array_equal(host(wdev[l]).ravel().view(np.uint32), upd[l]["w"].view(np.uint32)), l
        assert np.array_equal(host(net.tensor(l, pkg.NT_QW)).astype(np.int64), upd[l]["q"]), l
        assert (st.nnz, st.saturated) == (upd[l]["nnz"], upd[l]["sat"]), l
        assert (st.range_lo, st.range_hi) == (np.float32(upd[l]["lo"]), np.float32(upd[l]["hi"])), l
    # a second forward pass runs on the updated codes
    net.forward(dev(x), seed=seed, stream=s0 + 500)
    wq2 = [u["q"].reshape(w.shape) for u, w in zip(upd, wq)]
    fwd2 = no.forward(layers, fmts, wq2, x, seed, s0 + 500)
    assert np.array_equal(host(net.tensor(last, pkg.NT_A)).astype(np.int64), fwd2["a"][last].ravel())
    net.close()


def _small_net():
    return [no.Layer(8, 8, 4, 8, relu=True, pool=True),
            no.Layer(4, 4, 8, 8, relu=True, pool=False),
            no.Layer(1, 1, 128, 10, 1, 1, 1, 0, relu=False, pool=False)]


@pytest.mark.parametrize("fmts", [[(8, 5), (8, 5), (8, 4)], [(8, 5), (12, 8), (6, 3)], [(16, 11), (4, 2), (12, 8)],
                                  [(12, 9), (16, 12), (16, 10)]])
def test_small_chain_all_tensors(fmts):
    _run_chain(_small_net(), fmts, n=5, seed=sum(w for w, _ in fmts))


def test_vgg_like_chain_with_wide_channels():
    layers = [no.Layer(16, 16, 16, 64, relu=True, pool=False),
              no.Layer(16, 16, 64, 64, relu=True, pool=True),
              no.Layer(8, 8, 64, 128, relu=True, pool=True),
              no.Layer(1, 1, 4 * 4 * 128, 256, 1, 1, 1, 0, relu=True, pool=False),
              no.Layer(1, 1, 256, 10, 1, 1, 1, 0, relu=False, pool=False)]
    _run_chain(layers, [(8, 5), (8, 5), (6, 4), (12, 8), (8, 4)], n=8, seed=21)


def test_deep_chain_updates_more_layers_than_one_batched_launch_holds():
    # 40 layers: the batched update takes 32 tensors per launch, the 33rd starts a second one; ragged weight counts
    # (24 x 24 and 24 x 10 elements) put the tails of several tensors into one launch
    layers = [no.Layer(1, 1, 24, 24, 1, 1, 1, 0, relu=(l % 3 != 2), pool=False) for l in range(39)]
    layers.append(no.Layer(1, 1, 24, 10, 1, 1, 1, 0, relu=False, pool=False))
    fmts = [((8, 4), (12, 8), (16, 11), (6, 3))[l % 4] for l in range(40)]
    _run_chain(layers, fmts, n=6, seed=77)


def test_more_gradient_blocks_than_the_maxima_buffer_of_the_step_holds():
    # 1.1 M output rows: the data gradient of the second layer runs 8800 blocks of 128 rows, more than the 8192 maxima the
    # step has room for, so the fitting pass finds the largest magnitude in a pass of its own
    layers = [no.Layer(32, 32, 16, 16, relu=True, pool=False), no.Layer(32, 32, 16, 16, relu=True, pool=True),
              no.Layer(1, 1, 16 * 16 * 16, 10, 1, 1, 1, 0, relu=False, pool=False)]
    _run_chain(layers, [(8, 5), (8, 5), (8, 4)], n=1100, seed=5)


def test_a_context_too_small_for_the_batched_calls_reports_it():
    # six layers with 3.4 M weights: the batched quantize and the batched update want 6 x 16 KiB of per-block partials
    # each (1024 blocks), more than this context's 64 KiB of scratch
    small = pkg.Context(workspace_bytes=64 << 10)
    shapes = [(256, 1024), (1024, 1024), (1024, 1024), (1024, 1024), (1024, 64), (64, 10)]
    descs = [LayerDesc(ConvDesc(4, 1, 1, c, k, 1, 1, 1, 0), int(k != 10), 0) for c, k in shapes]
    w = [dev(np.zeros((k, 1, 1, c), np.float32)) for c, k in shapes]
    net = pkg.Net(small, descs, w)
    with pytest.raises(pkg.AdaptError) as e:
        net.quantize_weights()
    assert e.value.status == -5                          # ADAPT_EWORKSPACE
    net.close()
    small.close()


def test_deep_chain_with_some_layers_above_sixteen_bits_updates_them_one_by_one():
    layers = [no.Layer(1, 1, 16, 16, 1, 1, 1, 0, relu=True, pool=False) for _ in range(34)]
    layers.append(no.Layer(1, 1, 16, 10, 1, 1, 1, 0, relu=False, pool=False))
    fmts = [((8, 4), (20, 14), (12, 8))[l % 3] for l in range(35)]
    _run_chain(layers, fmts, n=4, seed=78, wl_max=32)


def test_alexnet_cifar_chain_reduced_batch():
    layers, fmts = [], []
    for sp, relu, pool in wk.alexnet_cifar_chain(batch=2):
        s = sp.shape
        layers.append(no.Layer(s.h, s.w, s.c, s.k, s.r, s.s, s.stride, s.pad, relu=relu, pool=pool))
        fmts.append((sp.wl, sp.fl))
    _run_chain(layers, fmts, n=2, seed=4)


def test_invalid_chains_are_rejected():
    bad = [LayerDesc(ConvDesc(2, 8, 8, 4, 8, 3, 3, 1, 1), 1, 1), LayerDesc(ConvDesc(2, 8, 8, 8, 8, 3, 3, 1, 1), 1, 0)]   # 4x4 != 8x8
    w = [dev(np.zeros((8, 3, 3, 4), np.float32)), dev(np.zeros((8, 3, 3, 8), np.float32))]
    with pytest.raises(pkg.AdaptError):
        pkg.Net(ctx(), bad, w)
    odd = [LayerDesc(ConvDesc(2, 7, 7, 4, 8, 3, 3, 1, 1), 1, 1)]
    with pytest.raises(pkg.AdaptError):
        pkg.Net(ctx(), odd, w[:1])
    ok = [LayerDesc(ConvDesc(2, 8, 8, 4, 8, 3, 3, 1, 1), 1, 1)]
    net = pkg.Net(ctx(), ok, w[:1])
    with pytest.raises(pkg.AdaptError):                    # backward before any forward pass
        net.backward(dev(np.zeros((2, 4, 4, 8), np.int8)), 0)
    net.close()


# ---- the whole of Alg. 1 with the precision switch of Alg. 2 -----------------------------------------------

def _train_with_switch(layers, fmts, n, steps, seed, sp_kw, fl_jumps=None, cx=None, starved=None, used_seen=None, wl_max=16):
    """fl_jumps: step -> added to the fractional bits the loss gradient is declared with (its codes stay the same);
    cx: the context to run on; starved: an empty list: the first precision switch that fails for lack of scratch in cx
    is repeated after the scratch has grown, and its step is appended; used_seen: list that collects r.used."""
    from oracle import pushup_oracle as po
    rng = np.random.default_rng(seed)
    first = layers[0]
    ws = [(rng.standard_normal((L.k, L.r, L.s, L.c)) * (1.5 / np.sqrt(L.r * L.s * L.c))).astype(np.float32) for L in layers]
    descs = [LayerDesc(ConvDesc(n, L.h, L.w, L.c, L.k, L.r, L.s, L.stride, L.pad), int(L.relu), int(L.pool)) for L in layers]
    wdev = [dev(w.copy()) for w in ws]
    sp = pkg.SwitchParams(sp_kw["lb_lwr"], sp_kw["lb_upr"], sp_kw["lb_init"], sp_kw["r_lwr"], sp_kw["r_upr"], sp_kw["r_init"],
                          sp_kw["gamma"], sp_kw["eps"], sp_kw["buff"], sp_kw["wl_lo"], sp_kw["wl_hi"], po.ST_MIN)
    net = pkg.Net(cx if cx is not None else ctx(), descs, wdev, switch=sp, wl_max=wl_max)
    fmts = list(fmts)
    for l, (wl, fl) in enumerate(fmts):
        net.set_format(l, wl, fl)
    st = no.SwitchState(len(layers), sp_kw["lb_lwr"], sp_kw["lb_upr"], sp_kw["lb_init"], sp_kw["r_lwr"], sp_kw["r_upr"],
                        sp_kw["r_init"], sp_kw["gamma"], sp_kw["eps"], sp_kw["buff"], sp_kw["wl_lo"], sp_kw["wl_hi"], wl_cap=wl_max)
    net.quantize_weights(seed=seed, stream=5)
    wq = no.quantize_weights(layers, fmts, ws, seed, 5)
    last = len(layers) - 1
    switches = 0
    for step in range(steps):
        s0 = 1000 * (step + 1)
        x = rng.standard_normal((n, first.h, first.w, first.c)).astype(np.float32)
        net.forward(dev(x), seed=seed, stream=s0)
        fwd = no.forward(layers, fmts, wq, x, seed, s0)
        got_logits = host(net.tensor(last, pkg.NT_A)).astype(np.int64)
        assert np.array_equal(got_logits, fwd["a"][last].ravel()), step
        wl_last, fl_last = fmts[last]
        logits = fwd["a"][last].reshape(n, -1) / 2.0 ** fl_last
        e = np.exp(logits - logits.max(axis=1, keepdims=True))
        soft = e / e.sum(axis=1, keepdims=True)
        labels = rng.integers(0, soft.shape[1], n)
        loss = float(-np.mean(np.log(soft[np.arange(n), labels] + 1e-30)))
        soft[np.arange(n), labels] -= 1.0
        dl_fl = wl_last - 1 + (fl_jumps or {}).get(step, 0)           # gradient of the logits in [-1, 1): WL-1 fractional bits
        lim = 1 << (wl_last - 1)
        dl = np.clip(np.rint(soft * lim), -lim, lim - 1).astype(_dt(wl_last))
        net.backward(dev(dl), dl_fl, seed=seed, stream=s0)
        bwd = no.backward(layers, fmts, wq, fwd, dl, seed, s0)
        try:
            rep, strat = net.precision_switch(loss, seed=seed, stream=s0)
        except pkg.AdaptError as err:
            if starved is None or starved or "workspace" not in str(err):
                raise
            starved.append(step)
            cx.reserve_workspace(64 << 20)
            rep, strat = net.precision_switch(loss, seed=seed, stream=s0)
        with pytest.raises(pkg.AdaptError):                           # the gradients of one backward pass join the windows once
            net.precision_switch(loss, seed=seed, stream=s0)
        want = no.precision_switch(st, fmts, ws, bwd, dl_fl, loss, seed, s0)
        if used_seen is not None:
            used_seen.extend(r.used for r in rep)
        assert strat == st.strategy, step
        for l, (r, w) in enumerate(zip(rep, want)):
            if np.isfinite(w["ds"]):
                assert abs(r.ds - w["ds"]) <= 1e-12 * abs(w["ds"]), (step, l)
            else:
                assert not np.isfinite(r.ds)
            assert (r.lb, r.res, bool(r.switched), r.wl, r.fl, r.used) == (w["lb"], w["res"], w["switched"], w["wl"], w["fl"], w["used"]), (step, l)
            if w["switched"]:
                switches += 1
                assert (r.wl_min, r.fl_min) == (w["wl_min"], w["fl_min"]), (step, l)
        net.update(0.05, 1e-5, 1e-4, seed=seed, stream=s0)
        upd = no.update(layers, fmts, ws, bwd, 0.05, 1e-5, 1e-4, seed, s0)
        for l in range(len(layers)):
            assert np.array_equal(host(wdev[l]).ravel().view(np.uint32), upd[l]["w"].view(np.uint32)), (step, l)
            assert np.array_equal(host(net.tensor(l, pkg.NT_QW)).astype(np.int64), upd[l]["q"]), (step, l)
        ws = [u["w"].reshape(w.shape) for u, w in zip(upd, ws)]
        wq = [u["q"].reshape(w.shape) for u, w in zip(upd, ws)]
    net.close()
    return switches, fmts


def test_training_steps_with_precision_switching_follow_the_oracle():
    kw = dict(lb_lwr=2, lb_upr=4, lb_init=2, r_lwr=50, r_upr=60, r_init=55, gamma=0.5, eps=1e-2, buff=2, wl_lo=2, wl_hi=16)
    switches, fmts = _train_with_switch(_small_net(), [(8, 5), (8, 5), (8, 4)], n=6, steps=8, seed=31, sp_kw=kw)
    assert switches >= 3


# ---- chains laid out for word lengths up to 32 ---------------------------------------------------------------

def _tiny_net():
    return [no.Layer(6, 6, 3, 8, relu=True, pool=True),
            no.Layer(3, 3, 8, 8, relu=True, pool=False),
            no.Layer(1, 1, 72, 5, 1, 1, 1, 0, relu=False, pool=False)]


@pytest.mark.parametrize("fmts", [[(24, 18), (20, 14), (32, 24)], [(8, 5), (24, 16), (12, 8)], [(17, 12), (16, 11), (17, 10)],
                                  [(32, 26), (32, 26), (32, 26)], [(12, 8), (8, 5), (8, 4)]])
def test_small_chain_with_layers_above_sixteen_bits(fmts):
    _run_chain(_tiny_net(), fmts, n=3, seed=sum(w for w, _ in fmts), wl_max=32)


@pytest.mark.parametrize("start,buff,eps,crossed", [([(14, 10), (20, 15), (8, 4)], 4, 1e-4, 1), ([(16, 12), (30, 24), (12, 8)], 6, 1e-6, 3)])
def test_training_steps_with_precision_switching_up_to_thirty_two_bits(start, buff, eps, crossed):
    # the second case takes a 16-bit and a 12-bit layer above 16 bits by PushUp and a 30-bit layer down to 21
    kw = dict(lb_lwr=2, lb_upr=3, lb_init=2, r_lwr=50, r_upr=60, r_init=55, gamma=0.5, eps=eps, buff=buff, wl_lo=2, wl_hi=32)
    switches, fmts = _train_with_switch(_tiny_net(), start, n=3, steps=7, seed=41, sp_kw=kw, wl_max=32)
    assert switches >= 6 and sum(w > 16 for w, _ in fmts) == crossed


def test_wide_chain_limits():
    descs = [LayerDesc(ConvDesc(2, 8, 8, 4, 8, 3, 3, 1, 1), 1, 1)]
    w = [dev(np.zeros((8, 3, 3, 4), np.float32))]
    net = pkg.Net(ctx(), descs, w)
    with pytest.raises(pkg.AdaptError):                    # a chain laid out for 16 bits takes no wider format
        net.set_format(0, 17, 12)
    net.close()
    net = pkg.Net(ctx(), descs, w, wl_max=32)
    net.set_format(0, 32, 20)
    with pytest.raises(pkg.AdaptError):
        net.set_format(0, 33, 20)
    net.close()
    with pytest.raises(pkg.AdaptError):
        pkg.Net(ctx(), descs, w, wl_max=24)


def test_precision_switching_across_the_one_and_two_limb_boundary():
    layers = [no.Layer(8, 8, 16, 32, relu=True, pool=True),
              no.Layer(4, 4, 32, 32, relu=True, pool=False),
              no.Layer(1, 1, 512, 16, 1, 1, 1, 0, relu=False, pool=False)]
    kw = dict(lb_lwr=1, lb_upr=3, lb_init=1, r_lwr=100, r_upr=128, r_init=100, gamma=0.3, eps=1e-3, buff=3, wl_lo=4, wl_hi=16)
    switches, fmts = _train_with_switch(layers, [(12, 9), (6, 3), (16, 12)], n=4, steps=6, seed=32, sp_kw=kw)
    assert switches >= 3


def test_gradient_scales_too_far_apart_drop_the_oldest_window_entries():
    # the declared scale of the loss gradient jumps by 2^40 between batches: a window that spans the jump cannot be
    # summed in 32 bits, so the entries before it are left out of the diversity (the oracle applies the same rule)
    kw = dict(lb_lwr=3, lb_upr=5, lb_init=4, r_lwr=50, r_upr=60, r_init=55, gamma=0.2, eps=1e-2, buff=2, wl_lo=2, wl_hi=16)
    used = []
    _train_with_switch(_small_net(), [(8, 5), (12, 8), (8, 4)], n=6, steps=7, seed=33, sp_kw=kw,
                       fl_jumps={2: 40, 3: 40, 4: 40, 5: -20, 6: -20}, used_seen=used)
    per_step = [used[i:i + 3] for i in range(0, len(used), 3)]
    assert any(u == 1 for u in per_step[2]) and any(u > 1 for row in per_step for u in row), per_step


@pytest.mark.parametrize("fmts", [[(8, 5), (12, 8)], [(10, 6), (8, 4)]])
def test_precision_switching_of_a_layer_whose_short_window_takes_several_chunks(fmts):
    # 2,113,536 weights: more than 1024 chunks of 2048, windows of one to three gradients (four chunks at a time) beside a
    # layer with one chunk per block
    layers = [no.Layer(1, 1, 2064, 1024, 1, 1, 1, 0, relu=True, pool=False), no.Layer(1, 1, 1024, 16, 1, 1, 1, 0, relu=False, pool=False)]
    kw = dict(lb_lwr=1, lb_upr=3, lb_init=3, r_lwr=50, r_upr=60, r_init=55, gamma=0.5, eps=1e-2, buff=2, wl_lo=6, wl_hi=10)
    used = []
    _train_with_switch(layers, fmts, n=4, steps=4, seed=35, sp_kw=kw, used_seen=used)
    assert max(used) >= 2, used


def test_a_precision_switch_that_fails_changes_nothing():
    # scratch that is enough for the contractions and the diversities but not for the KL search of a 64K-weight layer
    # at 4000 bins: the first call fails after the diversities were made, the repeated call must match the oracle,
    # and so must the steps after it (strategy, loss history, windows, lookbacks and formats were left alone)
    layers = [no.Layer(8, 8, 16, 32, relu=True, pool=True),
              no.Layer(4, 4, 32, 32, relu=True, pool=False),
              no.Layer(1, 1, 512, 128, 1, 1, 1, 0, relu=False, pool=False)]
    kw = dict(lb_lwr=1, lb_upr=3, lb_init=2, r_lwr=3000, r_upr=4096, r_init=4000, gamma=0.3, eps=1e-3, buff=3, wl_lo=4, wl_hi=16)
    cx = pkg.Context(workspace_bytes=1 << 20)
    try:
        starved = []
        switches, _ = _train_with_switch(layers, [(12, 9), (6, 3), (16, 12)], n=4, steps=5, seed=34, sp_kw=kw, cx=cx, starved=starved)
    finally:
        cx.close()
    assert switches >= 2 and len(starved) == 1 and starved[0] >= 1        # the loss history was in use when the call failed


def test_precision_switch_needs_a_backward_pass_and_parameters():
    ok = [LayerDesc(ConvDesc(2, 8, 8, 4, 8, 3, 3, 1, 1), 1, 1)]
    w = [dev(np.zeros((8, 3, 3, 4), np.float32))]
    net = pkg.Net(ctx(), ok, w)
    with pytest.raises(pkg.AdaptError):
        net.precision_switch(1.0)                         # created without switch parameters
    net.close()
    bad = pkg.SwitchParams(3, 2, 2, 50, 60, 55, 0.5, 1e-2, 2, 2, 16, 0)       # lb_lwr > lb_upr
    with pytest.raises(pkg.AdaptError):
        pkg.Net(ctx(), ok, w, switch=bad)
    good = pkg.SwitchParams(2, 4, 2, 50, 60, 55, 0.5, 1e-2, 2, 2, 16, 0)
    net = pkg.Net(ctx(), ok, w, switch=good)
    with pytest.raises(pkg.AdaptError):
        net.precision_switch(1.0)                         # no backward pass yet
    net.close()


# ---- random small chains: narrow first layers, stride 2, mixed word lengths, pooling in any combination ---------

def _random_net(rng):
    h = w = int(rng.choice([8, 12, 16]))
    c = int(rng.choice([1, 3, 5, 16, 24]))
    layers, fmts = [], []
    nconv = int(rng.integers(2, 5))
    for i in range(nconv):
        k = int(rng.choice([8, 16, 32, 64]))
        r = int(rng.choice([1, 3]))
        stride = int(rng.choice([1, 1, 2])) if h % 2 == 0 and h >= 8 else 1
        pad = r // 2
        L = no.Layer(h, w, c, k, r, r, stride, pad, relu=bool(rng.integers(0, 4) > 0), pool=False)
        p, q = L.p, L.q
        if p % 2 == 0 and q % 2 == 0 and p >= 4 and rng.integers(0, 3) == 0:
            L.pool = True
            p, q = p // 2, q // 2
        layers.append(L)
        fmts.append((int(rng.choice([4, 6, 8, 8, 11, 14, 16])), 0))
        h, w, c = p, q, k
    layers.append(no.Layer(1, 1, h * w * c, int(rng.choice([10, 16, 100])), 1, 1, 1, 0, relu=False, pool=False))
    fmts.append((int(rng.choice([6, 8, 12, 16])), 0))
    fmts = [(wl, wl - 3) for wl, _ in fmts]
    return layers, fmts


@pytest.mark.parametrize("seed", range(8))
def test_random_chains(seed):
    rng = np.random.default_rng(1000 + seed)
    layers, fmts = _random_net(rng)
    _run_chain(layers, fmts, n=int(rng.choice([2, 3, 5])), seed=100 + seed)


def test_alexnet_chain_full_batch_forward_matches_the_oracle_on_its_first_samples():
    """Batch 128 is the size the benchmark times (other tiles, K splits and launch shapes than the small cases).  The
    forward pass treats samples independently and a sample's rounding bits depend only on its element indices, so the
    first samples of the full batch must equal the oracle's forward pass on those samples alone."""
    batch, sub = 128, 2
    rng = np.random.default_rng(77)
    layers, fmts, descs = [], [], []
    for sp, relu, pool in wk.alexnet_cifar_chain(batch=batch):
        s = sp.shape
        layers.append(no.Layer(s.h, s.w, s.c, s.k, s.r, s.s, s.stride, s.pad, relu=relu, pool=pool))
        descs.append(LayerDesc(ConvDesc(batch, s.h, s.w, s.c, s.k, s.r, s.s, s.stride, s.pad), int(relu), int(pool)))
        fmts.append((sp.wl, sp.fl))
    x = rng.standard_normal((batch, 32, 32, 3)).astype(np.float32)
    ws = [(rng.standard_normal((L.k, L.r, L.s, L.c)) * (1.5 / np.sqrt(L.r * L.s * L.c))).astype(np.float32) for L in layers]
    big = ctx()
    big.reserve_for_layers([(d.conv, f, f, f) for d in descs for f in ((8, 5), (16, 13))])
    net = pkg.Net(big, descs, [dev(w) for w in ws])
    for l, (wl, fl) in enumerate(fmts):
        net.set_format(l, wl, fl)
    net.quantize_weights(seed=5, stream=9)
    net.forward(dev(x), seed=5, stream=9)
    wq = no.quantize_weights(layers, fmts, ws, 5, 9)
    fwd = no.forward(layers, fmts, wq, x[:sub], 5, 9)
    for l, L in enumerate(layers):
        got = host(net.tensor(l, pkg.NT_A)).astype(np.int64).reshape(L.out_shape(batch))[:sub]
        assert np.array_equal(got, fwd["a"][l]), l
    net.close()


# ---- the chain at the batch the benchmark times, every tensor against the oracle --------------------------------------
#
# Batch 128 takes other tiles, K splits and launch shapes than the small chains above.  One GPU step (forward,
# backward, update) is run once and its tensors kept on the host; the oracle's step is computed stage by stage, each
# test comparing one stage in full (every element of every tensor, all 128 samples).

_A128 = {}


def _alexnet128_gpu():
    if "gpu" in _A128:
        return _A128["gpu"]
    batch, seed, s0 = 128, 6, 4000
    rng = np.random.default_rng(78)
    layers, fmts, descs = [], [], []
    for sp, relu, pool in wk.alexnet_cifar_chain(batch=batch):
        s = sp.shape
        layers.append(no.Layer(s.h, s.w, s.c, s.k, s.r, s.s, s.stride, s.pad, relu=relu, pool=pool))
        descs.append(LayerDesc(ConvDesc(batch, s.h, s.w, s.c, s.k, s.r, s.s, s.stride, s.pad), int(relu), int(pool)))
        fmts.append((sp.wl, sp.fl))
    x = rng.standard_normal((batch, 32, 32, 3)).astype(np.float32)
    ws = [(rng.standard_normal((L.k, L.r, L.s, L.c)) * (1.5 / np.sqrt(L.r * L.s * L.c))).astype(np.float32) for L in layers]
    c = ctx()
    # operand formats differ between neighbouring layers of a chain: room for every layer at either storage width
    c.reserve_for_layers([(d.conv, f, f, f) for d in descs for f in ((8, 5), (16, 13))])
    wdev = [dev(w.copy()) for w in ws]
    net = pkg.Net(c, descs, wdev)
    for l, (wl, fl) in enumerate(fmts):
        net.set_format(l, wl, fl)
    net.quantize_weights(seed=seed, stream=s0)
    net.forward(dev(x), seed=seed, stream=s0)
    nl = len(layers)
    g = {"layers": layers, "fmts": fmts, "x": x, "ws": ws, "seed": seed, "s0": s0, "batch": batch}
    g["a_in"] = host(net.tensor(0, pkg.NT_INPUT)).astype(np.int64)
    g["qw"] = [host(net.tensor(l, pkg.NT_QW)).astype(np.int64) for l in range(nl)]
    g["y"] = [host(net.tensor(l, pkg.NT_Y)).astype(np.int64) for l in range(nl)]
    g["a"] = [host(net.tensor(l, pkg.NT_A)).astype(np.int64) for l in range(nl)]
    # the loss gradient is a function of the logits the GPU produced; the forward test shows them equal to the oracle's
    wl_last, fl_last = fmts[-1]
    logits = g["a"][-1].reshape(batch, -1) / 2.0 ** fl_last
    e = np.exp(logits - logits.max(axis=1, keepdims=True))
    soft = e / e.sum(axis=1, keepdims=True)
    soft[np.arange(batch), rng.integers(0, soft.shape[1], batch)] -= 1.0
    lim = 1 << (wl_last - 1)
    g["dl"] = np.clip(np.rint(soft * (lim - 1)), -lim, lim - 1).astype(_dt(wl_last))
    net.backward(dev(g["dl"]), 0, seed=seed, stream=s0)
    g["g"] = [host(net.tensor(l, pkg.NT_G)).astype(np.int64) for l in range(nl)]
    g["dy"] = [host(net.tensor(l, pkg.NT_DY)).astype(np.int64) for l in range(nl)]
    g["da"] = [host(net.tensor(l, pkg.NT_DA)).astype(np.int64) if l < nl - 1 else None for l in range(nl)]
    g["stats_bwd"] = [(st.shift_w, st.shift_a, st.g_sumsq) for st in (net.tensor(l, pkg.NT_STATS) for l in range(nl))]
    net.update(0.05, 1e-4, 1e-3, seed=seed, stream=s0)
    g["w_new"] = [host(w).ravel().view(np.uint32).copy() for w in wdev]
    g["qw_new"] = [host(net.tensor(l, pkg.NT_QW)).astype(np.int64) for l in range(nl)]
    g["stats_upd"] = [(st.nnz, st.saturated, st.range_lo, st.range_hi) for st in (net.tensor(l, pkg.NT_STATS) for l in range(nl))]
    net.close()
    _A128["gpu"] = g
    return g


def _alexnet128_oracle_fwd():
    if "fwd" not in _A128:
        g = _alexnet128_gpu()
        _A128["wq"] = no.quantize_weights(g["layers"], g["fmts"], g["ws"], g["seed"], g["s0"])
        _A128["fwd"] = no.forward(g["layers"], g["fmts"], _A128["wq"], g["x"], g["seed"], g["s0"])
    return _A128["wq"], _A128["fwd"]


def _alexnet128_oracle_bwd():
    if "bwd" not in _A128:
        g = _alexnet128_gpu()
        wq, fwd = _alexnet128_oracle_fwd()
        _A128["bwd"] = no.backward(g["layers"], g["fmts"], wq, fwd, g["dl"], g["seed"], g["s0"])
    return _A128["bwd"]


def test_alexnet_chain_full_batch_forward_in_full():
    g = _alexnet128_gpu()
    wq, fwd = _alexnet128_oracle_fwd()
    assert np.array_equal(g["a_in"], fwd["a_in"].ravel())
    for l in range(len(g["layers"])):
        assert np.array_equal(g["qw"][l], wq[l].ravel()), l
        assert np.array_equal(g["y"][l], fwd["y"][l].ravel()), l
        assert np.array_equal(g["a"][l], fwd["a"][l].ravel()), l


def test_alexnet_chain_full_batch_backward_in_full():
    g = _alexnet128_gpu()
    bwd = _alexnet128_oracle_bwd()
    for l, L in enumerate(g["layers"]):
        shift_w, shift_a, sumsq = g["stats_bwd"][l]
        assert np.array_equal(g["g"][l], bwd["g"][l].ravel()), l
        assert (shift_w, sumsq) == (bwd["shift_w"][l], bwd["sumsq"][l]), l
        if L.relu or L.pool:
            assert np.array_equal(g["dy"][l], bwd["dy"][l].ravel()), l
        if l > 0:
            assert shift_a == bwd["shift_a"][l], l
            assert np.array_equal(g["da"][l - 1], bwd["da"][l - 1].ravel()), l


@pytest.mark.parametrize("l", range(8))
def test_alexnet_chain_full_batch_update_in_full(l):
    from oracle import sgd_oracle as so
    g = _alexnet128_gpu()
    bwd = _alexnet128_oracle_bwd()
    wl, fl = g["fmts"][l]
    u = so.sgd_update_quantize(g["ws"][l].ravel(), bwd["g"][l].ravel(), 0, 0.05, 1e-4, 1e-3, wl, fl, orc.SR, g["seed"],
                               no.stream_of(g["s0"], l, no.SLOT_UPD), normalize=True)
    assert np.array_equal(g["w_new"][l], u["w"].view(np.uint32)), l
    assert np.array_equal(g["qw_new"][l], u["q"]), l
    nnz, sat, lo, hi = g["stats_upd"][l]
    assert (nnz, sat) == (u["nnz"], u["sat"]) and (lo, hi) == (np.float32(u["lo"]), np.float32(u["hi"])), l


# ---- residual networks with batch normalisation (the ResNets of Sec. 4.1) ------------------------------------------

from oracle import graph_oracle as go                                                   # noqa: E402
from paper_2107_13490_amd import NodeDesc                                               # noqa: E402


def _node_desc(n, L):
    return NodeDesc(ConvDesc(n, L.h, L.w, L.c, L.k, L.r, L.s, L.stride, L.pad), int(L.relu), int(L.pool), int(L.bn), L.src, L.res,
                    int(L.gap))


def _small_resnet():
    N = go.Node
    return [N(8, 8, 3, 8, bn=True),                                              # 0 stem
            N(8, 8, 8, 8, bn=True),                                              # 1 block A conv1
            N(8, 8, 8, 8, bn=True, res=0),                                       # 2 block A conv2 + identity
            N(8, 8, 8, 16, stride=2, bn=True, src=2),                            # 3 block B conv1 (stride 2)
            N(8, 8, 8, 16, 1, 1, 2, 0, relu=False, bn=True, src=2),              # 4 block B projection 1x1 stride 2
            N(4, 4, 16, 16, bn=True, src=3, res=4, gap=True),                    # 5 block B conv2 + projection, then pooling
            N(1, 1, 16, 10, 1, 1, 1, 0, relu=False)]                             # 6 fully connected


def _tiny_resnet():
    """The same topology on 4x4 maps (the oracle above 16 bits runs on Python integers)."""
    N = go.Node
    return [N(4, 4, 3, 8, bn=True),
            N(4, 4, 8, 8, bn=True),
            N(4, 4, 8, 8, bn=True, res=0),
            N(4, 4, 8, 16, stride=2, bn=True, src=2),
            N(4, 4, 8, 16, 1, 1, 2, 0, relu=False, bn=True, src=2),
            N(2, 2, 16, 16, bn=True, src=3, res=4, gap=True),
            N(1, 1, 16, 10, 1, 1, 1, 0, relu=False)]


def _resnet18_cifar(classes=100):
    N = go.Node
    nodes = [N(32, 32, 3, 64, bn=True)]
    cin, res, last = 64, 32, 0
    for stage, cout in enumerate([64, 128, 256, 512]):
        for block in range(2):
            stride = 2 if (stage > 0 and block == 0) else 1
            inp = last
            nodes.append(N(res, res, cin, cout, 3, 3, stride, 1, bn=True, src=inp))
            c1 = len(nodes) - 1
            short = inp
            if stride == 2:
                nodes.append(N(res, res, cin, cout, 1, 1, 2, 0, relu=False, bn=True, src=inp))
                short = len(nodes) - 1
                res //= 2
            final = stage == 3 and block == 1
            nodes.append(N(res, res, cout, cout, 3, 3, 1, 1, bn=True, src=c1, res=short, gap=final))
            last = len(nodes) - 1
            cin = cout
    nodes.append(N(1, 1, 512, classes, 1, 1, 1, 0, relu=False))
    return nodes


def _bn_state(net, l, k):
    raw = host(net.tensor(l, pkg.NT_BN))
    hdr = raw[:64].view(np.int32)
    body = raw[64:]
    return {"FA": int(hdr[3]), "FB": int(hdr[4]), "mean": body[:8 * k].view(np.float64), "A": body[40 * k:44 * k].view(np.int32),
            "B": body[24 * k:32 * k].view(np.int64)}


def _graph_step(net, nodes, fmts, ws, wdev, bn, bndev, x, labels_rng, seed, s0, lr, check_all, sw=None, forward_only=False):
    """One training step on both sides, compared tensor by tensor.  Returns (new ws, new wq, new bn, loss)."""
    n = x.shape[0]
    last = len(nodes) - 1
    wq = sw["wq"]
    net.forward(dev(x), seed=seed, stream=s0)
    fwd = go.forward(nodes, fmts, wq, bn, x, 1e-5, seed, s0)
    for l, L in enumerate(nodes):
        if check_all or l == last:
            if L.bn:
                assert np.array_equal(host(net.tensor(l, pkg.NT_YC)).astype(np.int64), fwd["yc"][l].ravel()), l
                st = _bn_state(net, l, L.k)
                assert st["FA"] == fwd["bn"][l]["FA"] and np.array_equal(st["A"], fwd["bn"][l]["A"]) and np.array_equal(st["B"], fwd["bn"][l]["B"]), l
            assert np.array_equal(host(net.tensor(l, pkg.NT_Y)).astype(np.int64), fwd["y"][l].ravel()), l
            assert np.array_equal(host(net.tensor(l, pkg.NT_A)).astype(np.int64), fwd["a"][l].ravel()), l
    if forward_only:
        return ws, bn, 0.0
    wl_last, fl_last = fmts[last]
    logits = fwd["a"][last].reshape(n, -1) / 2.0 ** fl_last
    e = np.exp(logits - logits.max(axis=1, keepdims=True))
    soft = e / e.sum(axis=1, keepdims=True)
    labels = labels_rng.integers(0, soft.shape[1], n)
    loss = float(-np.mean(np.log(soft[np.arange(n), labels] + 1e-30)))
    soft[np.arange(n), labels] -= 1.0
    dl_fl = wl_last - 1
    lim = 1 << (wl_last - 1)
    dl = np.clip(np.rint(soft * lim), -lim, lim - 1).astype(_dt(wl_last))
    net.backward(dev(dl), dl_fl, seed=seed, stream=s0)
    bwd = go.backward(nodes, fmts, wq, fwd, dl, dl_fl, seed, s0)
    for l, L in enumerate(nodes):
        ex = host(net.tensor(l, pkg.NT_EXP))
        assert np.array_equal(host(net.tensor(l, pkg.NT_G)).astype(np.int64), bwd["g"][l].ravel()), l
        assert int(ex[2]) == bwd["e_g"][l], (l, ex, bwd["e_g"][l])
        st_l = net.tensor(l, pkg.NT_STATS)
        assert (_sumsq(st_l) if fmts[l][0] > 16 else st_l.g_sumsq) == bwd["sumsq"][l], l
        if check_all:
            if l < last or L.bn or L.relu or L.pool:             # (the last layer may use the caller's gradient as it is)
                assert np.array_equal(host(net.tensor(l, pkg.NT_DYC)).astype(np.int64), bwd["dyc"][l].ravel()), l
            if l < last:
                assert np.array_equal(host(net.tensor(l, pkg.NT_DA)).astype(np.int64), bwd["da"][l].ravel()), l
                assert int(ex[0]) == bwd["e_da"][l], l
        if L.bn:
            assert np.array_equal(host(net.tensor(l, pkg.NT_DGAMMA)).view(np.uint64), bwd["dgamma"][l].view(np.uint64)), l
            assert np.array_equal(host(net.tensor(l, pkg.NT_DBETA)).view(np.uint64), bwd["dbeta"][l].view(np.uint64)), l
    if sw is not None and sw.get("state") is not None:
        rep, strat = net.precision_switch(loss, seed=seed, stream=s0)
        want = no.precision_switch(sw["state"], fmts, ws, bwd, dl_fl, loss, seed, s0)
        assert strat == sw["state"].strategy
        for l, (r, w) in enumerate(zip(rep, want)):
            if np.isfinite(w["ds"]):
                assert abs(r.ds - w["ds"]) <= 1e-12 * abs(w["ds"]), l
            assert (r.lb, r.res, bool(r.switched), r.wl, r.fl, r.used) == (w["lb"], w["res"], w["switched"], w["wl"], w["fl"], w["used"]), l
            sw["switches"] += int(w["switched"])
    net.update(lr, 1e-5, 1e-4, seed=seed, stream=s0)
    upd, bn_new = go.update(nodes, fmts, ws, bn, bwd, lr, 1e-5, 1e-4, seed, s0)
    for l, L in enumerate(nodes):
        assert np.array_equal(host(wdev[l]).ravel().view(np.uint32), upd[l]["w"].view(np.uint32)), l
        assert np.array_equal(host(net.tensor(l, pkg.NT_QW)).astype(np.int64), upd[l]["q"]), l
        if L.bn:
            assert np.array_equal(host(bndev[l][0]).view(np.uint32), bn_new[l][0].view(np.uint32)), l
            assert np.array_equal(host(bndev[l][1]).view(np.uint32), bn_new[l][1].view(np.uint32)), l
    ws = [u["w"].reshape(w.shape) for u, w in zip(upd, ws)]
    sw["wq"] = [u["q"].reshape(w.shape) for u, w in zip(upd, ws)]
    return ws, bn_new, loss


def _run_graph(nodes, fmts, n, steps, seed, switch_kw=None, check_all=True, lr=0.05, wl_max=16, forward_only=False):
    from oracle import pushup_oracle as po
    rng = np.random.default_rng(seed)
    first = nodes[0]
    ws = [(rng.standard_normal((L.k, L.r, L.s, L.c)) * (1.4 / np.sqrt(L.r * L.s * L.c))).astype(np.float32) for L in nodes]
    bn = [((1.0 + 0.2 * rng.standard_normal(L.k)).astype(np.float32), (0.1 * rng.standard_normal(L.k)).astype(np.float32)) if L.bn else None
          for L in nodes]
    wdev = [dev(w.copy()) for w in ws]
    bndev = [(dev(p[0].copy()), dev(p[1].copy())) if p else None for p in bn]
    sp = None
    state = None
    if switch_kw:
        k = switch_kw
        sp = pkg.SwitchParams(k["lb_lwr"], k["lb_upr"], k["lb_init"], k["r_lwr"], k["r_upr"], k["r_init"], k["gamma"], k["eps"], k["buff"],
                              k["wl_lo"], k["wl_hi"], po.ST_MIN)
        state = no.SwitchState(len(nodes), k["lb_lwr"], k["lb_upr"], k["lb_init"], k["r_lwr"], k["r_upr"], k["r_init"], k["gamma"], k["eps"],
                               k["buff"], k["wl_lo"], k["wl_hi"], wl_cap=wl_max)
    net = pkg.Net(ctx(), [_node_desc(n, L) for L in nodes], wdev, switch=sp, bn=bndev, bn_eps=1e-5, wl_max=wl_max)
    fmts = list(fmts)
    for l, (wl, fl) in enumerate(fmts):
        net.set_format(l, wl, fl)
    net.quantize_weights(seed=seed, stream=5)
    sw = {"wq": no.quantize_weights(nodes, fmts, ws, seed, 5), "state": state, "switches": 0}
    for step in range(steps):
        x = rng.standard_normal((n, first.h, first.w, first.c)).astype(np.float32)
        for l, (wl, fl) in enumerate(fmts):                      # formats may have switched
            pass
        ws, bn, _ = _graph_step(net, nodes, fmts, ws, wdev, bn, bndev, x, rng, seed, 1000 * (step + 1), lr, check_all, sw, forward_only)
    net.close()
    return sw["switches"], fmts


@pytest.mark.parametrize("fmts", [[(8, 4)] * 7, [(12, 8), (8, 4), (16, 11), (6, 3), (12, 7), (8, 4), (12, 8)],
                                  [(16, 12), (16, 11), (8, 5), (12, 8), (8, 3), (16, 11), (6, 2)]])
def test_small_residual_network_all_tensors(fmts):
    _run_graph(_small_resnet(), fmts, n=6, steps=2, seed=41)


def test_residual_network_whose_fitted_gradient_holds_the_most_negative_code():
    # in the second step the data gradient handed to layer 3 (7 bits) contains -64: stored as the fitting pass wrote it
    fmts = [(9, 5), (5, 2), (14, 9), (7, 4), (5, 0), (10, 7), (13, 9)]
    _run_graph(_small_resnet(), fmts, n=4, steps=2, seed=1711)


def test_residual_network_training_with_precision_switching():
    kw = dict(lb_lwr=1, lb_upr=3, lb_init=2, r_lwr=50, r_upr=80, r_init=60, gamma=0.4, eps=1e-2, buff=3, wl_lo=4, wl_hi=16)
    switches, fmts = _run_graph(_small_resnet(), [(12, 8)] * 6 + [(12, 7)], n=6, steps=6, seed=42, switch_kw=kw)
    assert switches >= 6


@pytest.mark.parametrize("fmts", [[(24, 18), (20, 14), (32, 25), (17, 11), (28, 20), (24, 17), (20, 14)],
                                  [(12, 8), (24, 18), (16, 11), (8, 4), (32, 24), (8, 4), (12, 8)]])
def test_small_residual_network_above_sixteen_bits(fmts):
    _run_graph(_tiny_resnet(), fmts, n=3, steps=2, seed=51, wl_max=32)


def test_residual_network_training_with_precision_switching_up_to_thirty_two_bits():
    kw = dict(lb_lwr=1, lb_upr=3, lb_init=2, r_lwr=50, r_upr=80, r_init=60, gamma=0.4, eps=1e-6, buff=6, wl_lo=4, wl_hi=32)
    switches, fmts = _run_graph(_tiny_resnet(), [(16, 12), (30, 24), (12, 8), (14, 10), (20, 15), (16, 11), (12, 7)], n=3, steps=5,
                                seed=52, switch_kw=kw, wl_max=32)
    assert switches >= 6 and sum(w > 16 for w, _ in fmts) >= 3


def test_graph_descriptions_that_are_rejected():
    w = [dev(np.zeros((8, 3, 3, 8), np.float32))] * 3
    p = [(dev(np.ones(8, np.float32)), dev(np.zeros(8, np.float32)))] * 3
    c = ConvDesc(2, 4, 4, 8, 8, 3, 3, 1, 1)
    bad = [[NodeDesc(c, 1, 0, 0, -1, 0, 0)],                                               # a shortcut without batch norm / from itself
           [NodeDesc(c, 1, 0, 1, -1, -1, 0), NodeDesc(c, 1, 0, 1, 1, -1, 0)],              # reads its own output
           [NodeDesc(c, 1, 0, 1, -1, -1, 0), NodeDesc(c, 1, 0, 1, -1, -1, 0), NodeDesc(c, 1, 0, 1, 0, -1, 0)],   # layer 1 has no consumer
           [NodeDesc(c, 1, 1, 1, -1, -1, 1)]]                                              # both kinds of pooling
    for nodes in bad:
        with pytest.raises(pkg.AdaptError):
            pkg.Net(ctx(), nodes, w[:len(nodes)], bn=p[:len(nodes)])
    with pytest.raises(pkg.AdaptError):                                                   # batch norm without its parameters
        pkg.Net(ctx(), [NodeDesc(c, 1, 0, 1, -1, -1, 0)], w[:1], bn=[None])


def _resnet18_formats(seed):
    g = np.random.default_rng(seed)
    fmts = [(int(wl), int(wl) - 4) for wl in g.integers(6, 17, 21)]
    fmts[0] = (12, 8)
    return fmts


def test_resnet18_cifar_chain_batch_64_every_tensor_of_a_step():
    # 4.2 M-element activations: every element-wise kernel runs several grid-stride rounds
    _run_graph(_resnet18_cifar(), _resnet18_formats(43), n=64, steps=1, seed=44, check_all=True, lr=0.02)


def test_resnet18_cifar_chain_full_batch_forward_every_tensor():
    # the batch the benchmark times (the whole step at this batch was compared once by hand: the oracle needs two minutes)
    _run_graph(_resnet18_cifar(), _resnet18_formats(43), n=256, steps=1, seed=45, check_all=True, forward_only=True)


def test_resnet18_cifar_chain_reduced_batch():
    nodes = _resnet18_cifar()
    g = np.random.default_rng(43)
    fmts = [(int(wl), int(wl) - 4) for wl in g.integers(8, 17, len(nodes))]
    fmts[0] = (12, 8)
    _run_graph(nodes, fmts, n=4, steps=1, seed=43, check_all=False, lr=0.02)


# ---- weight gradients with a short reduction, fitted without the exact sums in memory ------------------------------------
@pytest.mark.parametrize("batch,c,k,wl_x,wl_dy", [
    (128, 2000, 4080, 12, 13),      # whole stage; columns and rows that end inside a tile
    (1, 2048, 4096, 16, 16),        # offset split, one slot
    (127, 2000, 4096, 16, 16),
    (77, 2048, 4080, 8, 16),        # one int16 operand
    (77, 2048, 4080, 16, 5),
    (40, 2048, 4096, 7, 12),
    (40, 2048, 4096, 9, 8),
    (129, 1040, 1040, 8, 8),        # one limb: two stages per tile
    (256, 1024, 1024, 4, 8),
])
@pytest.mark.parametrize("kind", ["normal", "saturated", "one code"])
def test_fitted_weight_gradients_of_short_reductions(batch, c, k, wl_x, wl_dy, kind):
    g = np.random.default_rng(batch + c + k)
    ws = [g.standard_normal(16 * c).astype(np.float32), (0.01 * g.standard_normal(c * k)).astype(np.float32)]
    layers = [LayerDesc(ConvDesc(batch, 1, 1, 16, c, 1, 1, 1, 0), 0, 0), LayerDesc(ConvDesc(batch, 1, 1, c, k, 1, 1, 1, 0), 0, 0)]
    net = pkg.Net(ctx(), layers, [dev(w) for w in ws])
    # saturated inputs: sums at and next to powers of two, of either sign
    net.set_format(0, wl_x, max(0, wl_x - 4) if kind == "normal" else 0)
    net.set_format(1, wl_dy, 3)
    net.quantize_weights(seed=1)
    x = g.standard_normal((batch, 1, 1, 16)).astype(np.float32) * (1.0 if kind == "normal" else 3e4)
    net.forward(dev(x), seed=7, stream=50)
    lim = 1 << (wl_dy - 1)
    dl = g.integers(-lim, lim, (batch, k))
    if kind == "saturated":
        dl = g.choice([-lim, lim - 1, 0], (batch, k))
    elif kind == "one code":
        dl = np.zeros((batch, k), dtype=np.int64)
        dl[batch // 2, k - 1] = -1
    dl = dl.astype(_dt(wl_dy))
    net.backward(dev(dl), 0, seed=7, stream=50)
    a = host(net.tensor(0, pkg.NT_A)).reshape(batch, c)
    want, shift, sumsq = _fit_sums(a, dl, wl_dy, 7, 50 + 8 + 2)
    st = net.tensor(1, pkg.NT_STATS)
    assert (st.shift_w, _sumsq(st)) == (shift, sumsq)
    assert np.array_equal(host(net.tensor(1, pkg.NT_G)).astype(np.int64), want.ravel())


# ---- weight gradients on image rows whose launch, or whose slab sum, leaves the largest magnitude for the fit ----------------
ROWS_NETS = [
    # n, h, w, c, k, r, bits of the layer's inputs and of the layer, threads of the slab sum (0: none)
    (8, 16, 16, 512, 512, 3, 16, 16, 0),
    (8, 15, 17, 512, 496, 3, 12, 12, 0),
    (256, 4, 4, 512, 512, 3, 13, 12, 0),        # beside the data gradient
    (8, 16, 16, 512, 512, 3, 13, 8, 0),
    (8, 15, 17, 512, 496, 3, 16, 7, 0),
    (8, 16, 16, 512, 512, 3, 7, 16, 0),
    (8, 15, 17, 512, 496, 3, 8, 12, 0),
    (130, 16, 16, 128, 128, 3, 12, 12, 1),
    (130, 16, 16, 128, 128, 3, 8, 16, 1),
    (400, 32, 32, 64, 64, 1, 8, 12, 4),
    (400, 32, 32, 48, 48, 1, 12, 12, 16),
]


@pytest.mark.parametrize("case", ROWS_NETS)
def test_fitted_weight_gradients_on_image_rows(case):
    n, h, w, c, k, r, wl_x, wl_dy, _ = case
    g = np.random.default_rng(n + h + wl_x)
    conv = ConvDesc(n, h, w, c, k, r, 3, 1, 1)
    layers, ws = [LayerDesc(conv, 0, 0)], [(0.01 * g.standard_normal(c * k * r * 3)).astype(np.float32)]
    last = 0 if wl_x == wl_dy else 1
    if last:                                    # codes of another word length come from a layer in front
        layers.insert(0, LayerDesc(ConvDesc(n, h, w, 16, c, 1, 1, 1, 0), 0, 0))
        ws.insert(0, g.standard_normal(16 * c).astype(np.float32))
    net = pkg.Net(ctx(), layers, [dev(v) for v in ws])
    net.set_format(0, wl_x, max(0, wl_x - 4))
    if last:
        net.set_format(1, wl_dy, 3)
    net.quantize_weights(seed=1)
    net.forward(dev(g.standard_normal((n, h, w, 16 if last else c)).astype(np.float32)), seed=7, stream=50)
    lim = 1 << (wl_dy - 1)
    dl = g.choice([-lim, lim - 1, 0, 1, -1], (n, conv.p, conv.q, k)).astype(_dt(wl_dy))
    net.backward(dev(dl), 0, seed=7, stream=50)
    a = host(net.tensor(0, pkg.NT_A if last else pkg.NT_INPUT)).reshape(n, h, w, c)
    sums = co.conv_wgrad(dl, a, r, 3, 1, conv.pad)
    want, shift, sumsq = no.requantize_fit(sums.ravel(), wl_dy, orc.SR, 7, 50 + 8 * last + 2)
    st = net.tensor(last, pkg.NT_STATS)
    assert (st.shift_w, _sumsq(st)) == (shift, sumsq)
    assert np.array_equal(host(net.tensor(last, pkg.NT_G)).astype(np.int64), np.asarray(want).ravel())


def _fit_sums(a, dl, wl, seed, stream):
    # (float64 products of at most 2^30 each, at most 256 of them: exact)
    sums = (dl.astype(np.float64).T @ a.astype(np.float64)).astype(np.int64)
    shift = no.fit_shift(sums, wl)
    q = orc.requantize(sums, shift, wl, orc.SR, seed, stream, False)
    return q, shift, int((q * q).sum())
