"""Parity of the adjoint kernels (wm_predict_vjp, wm_loss_grad) and of the
autograd binding with the FP64 oracle gradient and with finite differences."""
import numpy as np
import pytest
import torch

from paper_2605_04178_amd import synth
from gpu_common import check_grad, loss_grad_absum, need_gpu, rel_err, say, slot_errors

pytestmark = pytest.mark.gpu
GTOL = 1e-4


@pytest.fixture(scope="module")
def wmb():
    need_gpu()
    from paper_2605_04178_amd import wavemodel
    wavemodel.lib()
    return wavemodel


def _measured(orc, p_true, d, sigma=0.02, seed=2):
    T, occ = orc.predict(p_true, d)
    return (T * synth.lognormal_noise(d.n, seed, sigma)).astype(np.float32)


@pytest.mark.parametrize("L,combine", [(4, 0), (3, 0), (4, 1)])
def test_loss_grad_parity_at_theta0(wmb, orc, L, combine):
    n = 1 << 18
    ps = synth.param_set(1, n_levels=L, combine=combine)
    d = synth.descriptors(n, 103)
    m = _measured(orc, ps, d)
    p0 = synth.perturb_theta(ps, 3)
    say("loss_grad parity", L, combine)
    dd = wmb.DeviceDescriptors.from_host(d)
    mt = torch.from_numpy(m).cuda()
    out = wmb.loss_grad(dd, mt, p0).cpu().numpy()
    loss, cnt, g = orc.loss_grad(p0, d, m)
    assert int(out[1]) == cnt
    assert abs(out[0] - loss) <= 1e-5 * loss
    check_grad(out[2:], g, p0.theta, f"loss gradient at theta0, L={L} combine={combine}", GTOL,
               names=synth.THETA_NAMES)


def test_loss_grad_parity_near_optimum(wmb, orc):
    """Close to theta*, |T/m - 1| is small for many descriptors, so the sign of
    each relative error is decided in FP64 where float32 cannot."""
    n = 1 << 18
    ps = synth.param_set(1)
    d = synth.descriptors(n, 104)
    m = _measured(orc, ps, d, sigma=0.02)
    dd = wmb.DeviceDescriptors.from_host(d)
    mt = torch.from_numpy(m).cuda()
    for k, f in enumerate((1.0, 1.001, 0.97)):
        p = ps.copy(theta=[t * (f if j % 3 == k else 1.0) for j, t in enumerate(ps.theta)])
        out = wmb.loss_grad(dd, mt, p).cpu().numpy()
        loss, cnt, g = orc.loss_grad(p, d, m)
        assert int(out[1]) == cnt
        assert abs(out[0] - loss) <= 1e-5 * loss
        check_grad(out[2:], g, p.theta, f"loss gradient near the optimum, factor {f} on slots {k} mod 3",
                   GTOL, names=synth.THETA_NAMES, absum=loss_grad_absum(orc, p, d, m))
        ex = wmb.loss_grad(dd, mt, p, exact=True).cpu().numpy()
        assert int(ex[1]) == cnt and abs(ex[0] - loss) <= 1e-12 * loss
        check_grad(ex[2:], g, p.theta, f"exact loss gradient near the optimum, factor {f}", GTOL,
                   names=synth.THETA_NAMES)


def test_loss_grad_exact_measurements(wmb, orc):
    """m = T(theta) exactly (noise-free): every relative error sits on the
    |.| kink; sign(0) = 0 must hold on both sides."""
    n = 1 << 16
    ps = synth.param_set(1)
    d = synth.descriptors(n, 105)
    T, _ = orc.predict(ps, d)
    m = T.astype(np.float32)
    dd = wmb.DeviceDescriptors.from_host(d)
    out = wmb.loss_grad(dd, torch.from_numpy(m).cuda(), ps).cpu().numpy()
    loss, cnt, g = orc.loss_grad(ps, d, m)
    assert int(out[1]) == cnt
    assert abs(out[0] - loss) <= 1e-5 * max(loss, 1e-12) + 1e-12
    check_grad(out[2:], g, ps.theta, "loss gradient with m = T", GTOL, names=synth.THETA_NAMES)


@pytest.mark.parametrize("L,combine", [(4, 0), (3, 1)])
def test_vjp_parity(wmb, orc, L, combine):
    n = 200003
    p = synth.param_set(0, n_levels=L, combine=combine)
    d = synth.descriptors(n, 106)
    w = np.random.default_rng(3).standard_normal(n).astype(np.float32)
    dd = wmb.DeviceDescriptors.from_host(d)
    g = wmb.vjp(dd, p, torch.from_numpy(w).cuda()).cpu().numpy()
    go = orc.vjp(p, d, w)
    check_grad(g, go, p.theta, f"vjp L={L} combine={combine}", GTOL, names=synth.THETA_NAMES)


def test_vjp_empty_and_deterministic(wmb):
    p = synth.param_set(0)
    d0 = wmb.DeviceDescriptors.from_host(synth.descriptors(0, 1))
    g0 = wmb.vjp(d0, p, torch.zeros(0, device="cuda"))
    assert torch.count_nonzero(g0).item() == 0
    dd = wmb.DeviceDescriptors.from_host(synth.descriptors(100000, 107))
    w = torch.randn(100000, device="cuda", generator=torch.Generator("cuda").manual_seed(1))
    a = wmb.vjp(dd, p, w)
    b = wmb.vjp(dd, p, w)
    assert torch.equal(a, b)


def test_autograd_function_matches_vjp_and_central_differences(wmb, orc):
    n = 1 << 18
    p = synth.param_set(0)
    d = synth.descriptors(n, 108)
    dd = wmb.DeviceDescriptors.from_host(d)
    theta = torch.tensor(p.theta, dtype=torch.float64, requires_grad=True)
    T = wmb.WMPredict.apply(dd, theta, p)
    fin = torch.isfinite(T)
    c = torch.from_numpy(np.random.default_rng(4).uniform(0.5, 1.5, n).astype(np.float32)).cuda()
    c = torch.where(fin, c, torch.zeros_like(c))
    L = (torch.where(fin, T, torch.zeros_like(T)).double() * c.double()).sum()
    L.backward()
    g = theta.grad.numpy()
    # equals the vjp call and the oracle's FP64 gradient
    gv = wmb.vjp(dd, p, c).cpu().numpy()
    assert np.array_equal(g, gv)
    go = orc.vjp(p, d, c.cpu().numpy())
    check_grad(g, go, p.theta, "autograd backward", GTOL, names=synth.THETA_NAMES)
    # central differences of the float32 forward sweep, h = 1e-4 relative
    h = 1e-4
    fd = np.zeros(24)
    for j in range(24):
        tp, tm = list(p.theta), list(p.theta)
        tp[j] *= 1 + h
        tm[j] *= 1 - h
        Tp, _ = wmb.predict(dd, p.copy(theta=tp), want_occ=False)
        Tm, _ = wmb.predict(dd, p.copy(theta=tm), want_occ=False)
        dp = (torch.where(fin, Tp, torch.zeros_like(Tp)).double() * c.double()).sum()
        dm = (torch.where(fin, Tm, torch.zeros_like(Tm)).double() * c.double()).sum()
        fd[j] = (dp - dm).item() / (2 * h * p.theta[j])
    # float32 forward values carry ~1e-7 relative rounding, which central
    # differences at h = 1e-4 turn into ~1e-3 of a slot's own term; slots
    # at 1e-2 of the largest log-space gradient or more are checked one by one
    ab, rel, big = slot_errors(fd, g, p.theta, floor=1e-2)
    say("finite differences vs autograd, per slot:", np.array2string(ab, precision=2),
        np.array2string(rel, precision=2))
    assert ab.max() <= 1e-3, (ab, fd, g)
    assert np.nanmax(rel) <= 3e-3, (rel, fd, g)


def test_loss_grad_workspace_reuse_and_determinism(wmb, orc):
    n = 300001
    ps = synth.param_set(1)
    d = synth.descriptors(n, 109)
    m = _measured(orc, ps, d)
    dd = wmb.DeviceDescriptors.from_host(d)
    mt = torch.from_numpy(m).cuda()
    ws = wmb._workspace(wmb.workspace_bytes(wmb.OP_LOSS_GRAD, n), "cuda")
    a = wmb.loss_grad(dd, mt, ps, ws=ws)
    b = wmb.loss_grad(dd, mt, ps, ws=ws)
    assert torch.equal(a, b)


@pytest.mark.parametrize("L,combine", [(4, 0), (3, 1)])
def test_exact_variants_match_the_oracle_slot_by_slot(wmb, orc, L, combine):
    """wm_predict_vjp_exact and wm_loss_grad_exact (float64 throughout the
    sweep) against the oracle, per slot in log space, at theta0 and at the
    true parameters (where the loss gradient is a cancelled sum)."""
    n = 1 << 18
    ps = synth.param_set(1, n_levels=L, combine=combine)
    d = synth.calibration_descriptors(n, 110)
    m = _measured(orc, ps, d)
    dd = wmb.DeviceDescriptors.from_host(d)
    mt = torch.from_numpy(m).cuda()
    for tag, p in (("theta0", synth.perturb_theta(ps, 3)), ("theta*", ps)):
        out = wmb.loss_grad(dd, mt, p, exact=True).cpu().numpy()
        loss, cnt, g = orc.loss_grad(p, d, m)
        assert int(out[1]) == cnt and abs(out[0] - loss) <= 1e-12 * loss
        check_grad(out[2:], g, p.theta, f"exact loss gradient at {tag}, L={L} combine={combine}", 1e-9,
                   names=synth.THETA_NAMES)
    w = np.random.default_rng(5).standard_normal(n).astype(np.float32)
    gv = wmb.vjp(dd, ps, torch.from_numpy(w).cuda(), exact=True).cpu().numpy()
    check_grad(gv, orc.vjp(ps, d, w), ps.theta, f"exact vjp, L={L} combine={combine}", 1e-9,
               names=synth.THETA_NAMES)


@pytest.mark.parametrize("n,block", [(1, 256), (64, 256), (960, 64), (16384, 64), (16448, 64), (20037, 128),
                                     (70001, 256), (131072, 64)])
def test_float64_pass_flags_and_row_slots(wmb, orc, n, block):
    """Every descriptor flagged (measured = the float64 time rounded to
    float32), so that the float64 pass's row queues overflow and refill, at
    its block-count edges (one block up to 16384 descriptors; block 64 with 960
    and 131072 leaves no row slot unused); nothing is written past the
    workspace.  All terms are float64: 1e-11 of each slot's absolute sum
    (a few thousand float64 roundings), and the loss, |T - m| / m ~ 1e-8
    formed from T to 1e-15, to 1e-13 absolute."""
    p = synth.param_set(6)
    d = synth.descriptors(n, 105)
    T, _ = orc.predict(p, d)
    m = np.where(np.isfinite(T), T, 1.0).astype(np.float32)
    loss, cnt, g = orc.loss_grad(p, d, m)
    absum = loss_grad_absum(orc, p, d, m)
    dd = wmb.DeviceDescriptors.from_host(d)
    need = wmb.workspace_bytes(wmb.OP_LOSS_GRAD, n)
    raw = torch.full((need + 512,), 0xAB, dtype=torch.uint8, device="cuda")
    off = (-raw.data_ptr()) % 256
    default = wmb.get_launch(wmb.OP_LOSS_GRAD, n)
    wmb.set_launch(wmb.OP_LOSS_GRAD, n, block, default["per_thread"], 8)
    try:
        say("float64 pass", n, block)
        out = wmb.loss_grad(dd, torch.from_numpy(m).cuda(), p, ws=raw[off:off + need]).cpu().numpy()
    finally:
        wmb.set_launch(wmb.OP_LOSS_GRAD, n, default["block"], default["per_thread"], default["grid_mult"])
    assert np.all(raw[off + need:].cpu().numpy() == 0xAB)
    assert int(out[1]) == cnt
    assert abs(out[0] - loss) <= 1e-13
    assert np.all(np.abs(out[2:] - g) * np.abs(p.theta) <= 1e-11 * absum + 1e-300)


def test_vjp_sweep_keeps_seven_waves_per_simd(wmb):
    """The adjoint sweep's partial rows in the workspace (26 doubles per block,
    then the float64 pass's and its count of finished blocks): seven blocks of 256
    per CU at 2^20 descriptors, whatever registers the kernel has."""
    n = 1 << 20
    p = synth.param_set(0)
    d = synth.descriptors(n, 106)
    w = np.random.default_rng(106).random(n).astype(np.float32)
    ws = torch.full((wmb.workspace_bytes(wmb.OP_VJP, n),), 0xAB, dtype=torch.uint8, device="cuda")
    assert ws.data_ptr() % 256 == 0
    wmb.vjp(wmb.DeviceDescriptors.from_host(d), p, torch.from_numpy(w).cuda(), ws=ws)
    first = ws[:26 * 8 * 4096].view(torch.int64).view(-1, 26)[:, 0].cpu().numpy()
    untouched = np.frombuffer(b"\xab" * 8, np.int64)[0]
    rows = int(np.argmax(first == untouched))
    words = n // 64
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    say("rows written", rows)
    assert rows == 7 * cus + words // 256 + 1


@pytest.mark.parametrize("n", [63, 65, 129, 257, 5000, 16321, 16385])
def test_float64_pass_of_one_block_shares_its_words(wmb, orc, n):
    """Every descriptor flagged, up to and past the 256 flag words that the four
    waves of a single block share: 1 to 5 words, shares that do not divide, the
    last word not full.  Tolerances as in the test of flags and row slots."""
    p = synth.param_set(6)
    d = synth.descriptors(n, 107)
    T, _ = orc.predict(p, d)
    m = np.where(np.isfinite(T), T, 1.0).astype(np.float32)
    loss, cnt, g = orc.loss_grad(p, d, m)
    out = wmb.loss_grad(wmb.DeviceDescriptors.from_host(d), torch.from_numpy(m).cuda(), p).cpu().numpy()
    assert int(out[1]) == cnt
    assert abs(out[0] - loss) <= 1e-13
    assert np.all(np.abs(out[2:] - g) * np.abs(p.theta) <= 1e-11 * loss_grad_absum(orc, p, d, m) + 1e-300)
