"""The paths a call takes by its sizes: each side of a dispatch rule against
the FP64 oracle, at the sizes where a rule or a remainder changes."""
import ctypes as C

import numpy as np
import pytest
import torch

from oracle import constraints as oc
from oracle.adam import adam_step
from paper_2505_07814_amd import _lib as L
from paper_2505_07814_amd import cnn, synth
from paper_2505_07814_amd.ptyr import AdamState, Engine
from test_gpu_cnn import make_case
from test_gpu_constraints import T, engine, rz_bound
from test_gpu_object_modes import ModeCase, _grad_errors
from test_gpu_parity import Case, _check_grads

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("S,H,W", [(1, 97, 130), (2, 353, 340)])
def test_scatter_tiles_and_more_than_64_rows(S, H, W):
    """Object gradient with 8-row tiles (few tiles) and 32-row tiles, over a
    batch of more rows than one wave tests at once; ragged object sides."""
    print(f"scatter S={S} H={H} W={W} B=67", flush=True)
    c = Case(synth.small_case(N=64, S=S, M=1, B=67, H=H, W=W, seed=41))
    _check_grads(c, c.engine())


@pytest.mark.parametrize("B,M,budget", [(3, 1, None), (130, 4, None), (6, 2, 0)])
def test_gradient_by_chains_per_compute_unit(B, M, budget):
    """N = 64 with few chains, with more than two chains per compute unit, and
    with no wave kept (the gradient recomputes them)."""
    print(f"gradient N=64 S=3 B={B} M={M} budget={budget}", flush=True)
    c = Case(synth.small_case(N=64, S=3, M=M, B=B, H=110, W=121, seed=43))
    _check_grads(c, c.engine(wave_budget=budget))


def test_gradient_between_one_and_two_chains_per_compute_unit():
    """N = 64: the forward with its twiddles in registers followed by the
    gradient without (one to two chains per compute unit), in one call and
    reusing the forward's waves."""
    B, M = 60, 5
    assert _units() < B * M <= 2 * _units()
    print(f"gradient N=64 S=3 B={B} M={M}", flush=True)
    c = Case(synth.small_case(N=64, S=3, M=M, B=B, H=110, W=121, seed=97))
    eng = c.engine()
    whole = _check_grads(c, eng)
    eng.forward(*c.gpu_args())
    reused = _check_grads(c, eng, reuse=True)
    # (the object's sums run over two ranges of rows in the first, over one in the second)
    assert all(torch.equal(whole[k], reused[k]) for k in ("probe", "pos", "tilt", "dz"))


@pytest.mark.parametrize("S,H,W,M", [(5, 64, 66, 2), (5, 65, 67, 7), (17, 64, 66, 24), (33, 64, 64, 3)])
def test_orthogonalisation_beside_the_depth_filter(S, H, W, M):
    """The eigen-solve inside the depth filter's launch (both filter kernels),
    after it (deep stacks), for odd and even numbers of modes."""
    print(f"rz + orthogonalisation S={S} {H}x{W} M={M}", flush=True)
    rng = np.random.default_rng(S * M)
    amp = rng.uniform(0.5, 1.5, (S, H, W)).astype(np.float32)
    ph = rng.uniform(-0.5, 1.0, (S, H, W)).astype(np.float32)
    scale = 1.0 / (1 + np.arange(M))[:, None, None]              # well-separated powers
    probe = (scale * (rng.standard_normal((M, 64, 64)) + 1j * rng.standard_normal((M, 64, 64)))).astype(np.complex64)
    eng = engine(S, H, W, 64, M)
    a, p, P = T(amp), T(ph), T(probe)
    eng.constrain(a, p, P, rz_sigma=1.0, phase_positive=True, probe_orthogonal=True)
    eng.sync()
    ra, rp, rP = oc.apply(amp, ph, probe, rz_sigma=1.0, phase_positive=True, probe_orthogonal=True)
    assert np.max(np.abs(a.cpu().numpy() - ra)) <= rz_bound(1.0, amp)
    assert np.max(np.abs(p.cpu().numpy() - rp)) <= rz_bound(1.0, ph)
    got = P.cpu().numpy()
    for m in range(M):                                           # up to each mode's unit phase
        u = np.vdot(got[m], rP[m])
        d = np.linalg.norm(got[m] * (u / abs(u)) - rP[m]) / np.linalg.norm(rP[m])
        assert d <= 1e-5, (m, d)


@pytest.mark.parametrize("bad", [np.nan, np.inf])
@pytest.mark.parametrize("S,M", [(5, 2), (5, 7), (33, 3)])
def test_orthogonalisation_of_a_bad_mode(S, M, bad):
    """A mode with one NaN pixel makes every mode NaN (none is dropped, doubled
    or left finite); one with an infinite pixel, whose power no overlap
    exceeds, leaves the modes as they are, largest power first, but for that
    pixel.  In the depth filter's launch and in its own; the filtered object of
    the same call is unaffected, and so is the next call."""
    print(f"orthogonalisation of a bad mode S={S} M={M} {bad}", flush=True)
    rng = np.random.default_rng(S + M)
    amp = rng.uniform(0.5, 1.5, (S, 64, 66)).astype(np.float32)
    ph = rng.uniform(-0.5, 1.0, (S, 64, 66)).astype(np.float32)
    good = (rng.standard_normal((M, 64, 64)) + 1j * rng.standard_normal((M, 64, 64))).astype(np.complex64)
    eng = engine(S, 64, 66, 64, M)
    for mode in (0, M - 1):
        probe = good.copy()
        probe[mode, 3, 5] = bad
        a, p, P = T(amp), T(ph), T(probe)
        eng.constrain(a, p, P, rz_sigma=1.0, phase_positive=True, probe_orthogonal=True)
        eng.sync()
        ra, rp, _ = oc.apply(amp, ph, good, rz_sigma=1.0, phase_positive=True, probe_orthogonal=True)
        assert np.max(np.abs(a.cpu().numpy() - ra)) <= rz_bound(1.0, amp)
        assert np.max(np.abs(p.cpu().numpy() - rp)) <= rz_bound(1.0, ph)
        got = P.cpu().numpy()
        if np.isnan(bad):
            assert np.all(np.isnan(got.real) & np.isnan(got.imag)), mode
        else:
            power = np.sum(np.abs(probe.astype(np.complex128)) ** 2, axis=(1, 2))
            keep = np.ones((64, 64), bool)
            keep[3, 5] = False
            assert np.array_equal(got[:, keep], probe[np.argsort(-power)][:, keep]), mode
            assert not np.isfinite(got[:, 3, 5]).any()
    P = T(good)
    eng.constrain(T(amp), T(ph), P, rz_sigma=1.0, probe_orthogonal=True)
    eng.sync()
    G = P.cpu().numpy().reshape(M, -1).astype(np.complex128)
    G = G.conj() @ G.T
    assert np.linalg.norm(G - np.diag(np.diag(G))) <= 1e-5 * np.linalg.norm(G)


@pytest.mark.parametrize("S,H,W", [(16, 96, 250), (24, 100, 640), (3, 64, 3375), (4, 3375, 64)])
def test_kz_filter_passes(S, H, W):
    """x and z in one pass and apart (by what fits a workgroup), radices 15,
    12, 10 and 9, padded pitches, a ragged last tile of columns."""
    print(f"kz passes {S}x{H}x{W}", flush=True)
    rng = np.random.default_rng(S + H + W)
    amp = rng.uniform(0.5, 1.5, (S, H, W)).astype(np.float32)
    ph = rng.uniform(-0.5, 1.0, (S, H, W)).astype(np.float32)
    eng = engine(S, H, W)
    a, p = T(amp), T(ph)
    eng.constrain(a, p, kz_beta=0.8, kz_alpha=0.5, kz_dz=5.0)
    eng.sync()
    for got, field in ((a, amp), (p, ph)):
        ref = oc.kz_filter(field, 0.8, 0.5, 0.2, 5.0)
        assert np.linalg.norm(got.cpu().numpy() - ref) <= 1e-5 * np.linalg.norm(ref)


@pytest.mark.parametrize("N,S,M,B", [(64, 3, 2, 5), (64, 3, 5, 110), (128, 3, 2, 3), (256, 2, 2, 2)])
def test_step_with_frozen_tilt_and_dz(N, S, M, B):
    """A step with tilts and dz frozen (no Y_s kept, no such sums) updates the
    other parameters exactly as one that also refines them, leaves tilts, dz
    and their moments alone, and a later gradient does not reuse its waves."""
    print(f"frozen tilt / dz N={N} S={S} M={M} B={B}", flush=True)
    c = Case(synth.small_case(N=N, S=S, M=M, B=B, H=N + 40, W=N + 47, seed=47), perturb=True)
    full = dict(amp=1e-3, phase=2e-3, probe=1e-2, pos=1e-2, tilt=1e-4, dz=1e-1)
    out = []
    for lr in (full, dict(full, tilt=0.0, dz=0.0)):
        eng = c.engine(n_scan=B)
        st = AdamState(*c.gpu_args())
        eng.step(st, T(np.arange(B, dtype=np.int32)), T(c.meas), lr)
        eng.sync()
        out.append((eng, st))
    (_, a), (eng, b) = out
    for k in ("amp", "phase", "probe", "pos"):
        assert torch.equal(getattr(a, k), getattr(b, k)), k
        assert torch.equal(a.m[k], b.m[k]) and torch.equal(a.v[k], b.v[k]), k
    assert np.array_equal(b.tilt.cpu().numpy(), c.tilt) and float(b.dz) == float(c.dz)
    assert not b.m["tilt"].any() and not b.v["dz"].any()
    args = tuple(getattr(b, k) for k in b.NAMES)
    l0, g0 = eng.adjoint(*args, T(c.meas), reuse=True)
    l1, g1 = eng.adjoint(*args, T(c.meas))
    eng.sync()
    assert all(torch.equal(g0[k], g1[k]) for k in g0) and torch.equal(l0, l1)


@pytest.mark.parametrize("M,B", [(8, 3), (3, 11), (5, 4), (8, 20)])
def test_gradient_256_row_groups(M, B):
    """N = 256 row pass: modes in groups of what leaves each compute unit a
    workgroup, by two halves of a workgroup (odd groups too) or by one."""
    print(f"gradient N=256 S=2 M={M} B={B}", flush=True)
    c = Case(synth.small_case(N=256, S=2, M=M, B=B, H=300, W=310, seed=53))
    _check_grads(c, c.engine())


def _units():
    return torch.cuda.get_device_properties(0).multi_processor_count


@pytest.mark.parametrize("S,M,B,two", [(12, 8, 2, True), (2, 8, 32, False)])
def test_gradient_256_groups_deep_and_in_one_half(S, M, B, two):
    """N = 256 row pass: a deep stack (every gradient, dz among them) with two
    halves per workgroup, and groups of 8 modes taken by one half, as they are
    from more than one workgroup of 16 lines per compute unit on."""
    assert (B * 16 <= _units()) == two
    print(f"gradient N=256 S={S} M={M} B={B} halves={1 + two}", flush=True)
    c = Case(synth.small_case(N=256, S=S, M=M, B=B, H=290, W=300, seed=79))
    _check_grads(c, c.engine())


@pytest.mark.parametrize("B,two", [(3, True), (16, False)])
def test_gradient_256_groups_of_two_object_modes(B, two):
    """Groups of probe modes stay within their object mode."""
    assert (2 * B * 16 <= _units()) == two
    print(f"gradient N=256 S=2 M=8 n_obj=2 B={B} halves={1 + two}", flush=True)
    c = ModeCase(256, 2, 8, B, seed=83, H=290, W=300)
    for k, e in _grad_errors(c, c.engine()).items():
        assert e < (1e-6 if k == "loss" else 1e-4), (k, e)


@pytest.mark.parametrize("which", ["one term", "all terms"])
def test_step_with_the_scatter_beside_the_reductions(which):
    """A one-stream N = 128 step whose object scatter moves enough to run on the
    side stream beside the probe's and parameters' reductions and Adam: the
    gradients of ptyr_adjoint followed by Adam in float64, over two steps (the
    second starts after the join)."""
    S, M, B = 7, 4, 40
    H, W = 180, 190
    assert B * M <= _units() and B * M * S * 128 * 128 * 8 + S * H * W * 48 >= 128e6
    print(f"step N=128 S={S} M={M} B={B}, {which}", flush=True)
    c = Case(synth.small_case(N=128, S=S, M=M, B=B, H=H, W=W, seed=89))
    lr = dict(amp=1e-3, phase=2e-3, probe=1e-2, pos=1e-2, tilt=1e-4, dz=1e-1)
    kw = dict(w_gaussian=0.7, w_poisson=0.4, pacbed_w=0.5, sparse_w=0.1) if which == "all terms" else {}
    eng, ref_eng = c.engine(n_scan=B, **kw), c.engine(**kw)
    st, meas = AdamState(*c.gpu_args()), T(c.meas)
    b1, b2, eps = (float(np.float32(x)) for x in (0.9, 0.999, 1e-8))
    real = lambda x: np.ravel(x.cpu().numpy()).view(np.float32).astype(np.float64)
    for t in range(2):
        idx = T(np.roll(np.arange(B, dtype=np.int32), t))
        before = [getattr(st, k).clone() for k in st.NAMES]
        m0, v0 = ({k: x[k].clone() for k in st.NAMES} for x in (st.m, st.v))
        loss = eng.step(st, idx, meas, lr).clone()
        ref_loss, g = ref_eng.adjoint(*before, meas, idx=idx)
        eng.sync()
        ref_eng.sync()
        assert torch.equal(loss, ref_loss)
        for k, old in zip(st.NAMES, before):
            p0 = real(old)
            want, _, _ = adam_step(p0, real(g[k]), real(m0[k]), real(v0[k]), t, lr[k], beta1=b1, beta2=b2, eps=eps)
            # the float32 parameter is the reference update rounded, to 2 ulp, and the update to float32 arithmetic
            tol = 2 * np.spacing(np.abs(want).astype(np.float32)) + 1e-5 * np.abs(want - p0)
            assert np.all(np.abs(real(getattr(st, k)) - want) <= tol), (t, k)


@pytest.mark.parametrize("B", [1, 2, 16, 32])
def test_object_gradient_256_adds_modes_in_order(B):
    """N = 256: the object gradient adds the probe modes of a group in mode
    order whatever the batch, and so whatever share of the chip the row pass
    has.  Modes 1 to 7 are the first times 2^-13, so every product of theirs is
    the first mode's times 2^-26 exactly and, added one by one, below a quarter
    unit in the last place: the intensities, the loss and the object gradient
    are bitwise those of the first mode alone.  Any partial sum of several
    small modes (four are half a unit) would round the result up."""
    print(f"object gradient order N=256 S=2 M=8 B={B}", flush=True)
    c = Case(synth.small_case(N=256, S=2, M=1, B=B, H=300, W=310, seed=59))
    args, meas = list(c.gpu_args()), T(c.meas)
    one = c.engine().adjoint(*args, meas)
    args[2] = torch.cat([args[2]] + 7 * [args[2] * 2.0 ** -13]).contiguous()
    eng = Engine(256, 8, 2, c.w.H, c.w.W, B, c.w.dx, c.lam, device=meas.device)
    eight = eng.adjoint(*args, meas)
    eng.sync()
    assert torch.equal(one[0], eight[0])
    assert float(torch.linalg.norm(one[1]["phase"])) > 0.0
    for k in ("amp", "phase"):
        assert torch.equal(one[1][k], eight[1][k]), k


def test_kz_filter_of_a_tiny_spacing():
    """A spacing so small that k_z^2 alone overflows float32 while the weight's
    beta^2 k_z^2 / (k_r^2 + 1e-3) stays below 1e-5: the filter leaves the object
    as it is."""
    print("kz filter, tiny spacing", flush=True)
    rng = np.random.default_rng(71)
    f = [rng.uniform(0.5, 1.5, (6, 64, 72)).astype(np.float32) for _ in range(2)]
    eng = engine(6, 64, 72)
    got = [T(x) for x in f]
    eng.constrain(*got, kz_beta=1e-25, kz_dz=1e-21)
    eng.sync()
    for g, x in zip(got, f):
        ref = oc.kz_filter(x, 1e-25, 0.0, 0.2, 1e-21)
        assert np.linalg.norm(g.cpu().numpy() - ref) <= 1e-5 * np.linalg.norm(ref)


def on_workspace(eng, ws):
    """The engine's context bound to `ws` instead of its own workspace."""
    lib, ctx = eng.lib, C.c_void_p()
    base = (ws.data_ptr() + 255) // 256 * 256
    assert base + eng._ws_bytes <= ws.data_ptr() + ws.numel()
    L.check(lib.ptyr_destroy(eng._ctx), "ptyr_destroy")
    L.check(lib.ptyr_create(C.byref(eng.geom), C.c_void_p(base), eng._ws_bytes, C.c_void_p(eng.stream.cuda_stream),
                            C.byref(ctx)), "ptyr_create")
    eng._ctx = ctx
    return eng


@pytest.mark.parametrize("N", [64, 128, 256])
def test_contexts_taking_turns_on_one_workspace(N):
    """A forward or a gradient forms all it reads from the workspace: contexts
    of two geometries on one workspace, overwritten between the calls, give
    bitwise the results of contexts with a workspace each."""
    print(f"shared workspace N={N}", flush=True)
    cases = [Case(synth.small_case(N=N, S=S, M=M, B=3, H=N + 40, W=N + 45, seed=61)) for S, M in ((2, 1), (3, 2))]
    ref = []
    for c in cases:
        eng = c.engine()
        ref.append((eng.forward(*c.gpu_args()).clone(), eng.adjoint(*c.gpu_args(), T(c.meas))))
        eng.sync()
    ws = torch.empty(max(c.engine()._ws_bytes for c in cases) + 256, dtype=torch.uint8, device="cuda:0")
    engines = [on_workspace(c.engine(), ws) for c in cases]
    for c, eng, (I, (loss, g)) in 2 * list(zip(cases, engines, ref)):
        ws.fill_(0xFF)
        assert torch.equal(eng.forward(*c.gpu_args()), I)
        ws.fill_(0xFF)
        loss2, g2 = eng.adjoint(*c.gpu_args(), T(c.meas))
        assert torch.equal(loss2, loss) and all(torch.equal(g2[k], g[k]) for k in g)
    torch.cuda.synchronize()


def test_constraints_on_a_shared_workspace():
    """The same for the constraints: k_z filter (x and z in one pass and apart),
    depth filter and eigen-solve form all they read in the call."""
    print("constraints on a shared workspace", flush=True)
    rng = np.random.default_rng(67)
    sizes = ((6, 96, 90), (24, 100, 640))
    ws = torch.empty(max(engine(*s, 64, 3)._ws_bytes for s in sizes) + 256, dtype=torch.uint8, device="cuda:0")
    kw = dict(rz_sigma=0.8, phase_positive=True, probe_orthogonal=True, kz_beta=0.8, kz_alpha=0.5, kz_dz=5.0)
    runs = []
    for S, H, W in sizes:
        f = [rng.uniform(0.5, 1.5, (S, H, W)).astype(np.float32) for _ in range(2)]
        f.append((rng.standard_normal((3, 64, 64)) + 1j * rng.standard_normal((3, 64, 64))).astype(np.complex64))
        own, out = engine(S, H, W, 64, 3), [T(x) for x in f]
        own.constrain(*out, **kw)
        runs.append((f, out, on_workspace(engine(S, H, W, 64, 3), ws)))
    for f, out, eng in 2 * runs:
        ws.fill_(0xFF)
        got = [T(x) for x in f]
        eng.constrain(*got, **kw)
        assert all(torch.equal(a, b) for a, b in zip(got, out))
    torch.cuda.synchronize()


@pytest.mark.parametrize("B", [2, 36])
def test_conv_net_gradient_is_the_mean_of_its_halves(B):
    """Weight gradients over fewer tiles than workgroups and (36 samples of 8
    tiles over 256 workgroups) over uneven shares: the gradient of a batch is
    the mean of those of its halves.  The output gradient differs by the exact
    factor 2, so every stored BF16 value scales exactly and only the order of
    float32 sums differs."""
    print(f"conv net gradient B={B}", flush=True)
    _, vec, pats, nbr, target = make_case(B, 40, 60 + B)
    net = cnn.ConvInit(B)
    V, P = T(vec), T(pats)

    def grad(sel):
        g = torch.zeros(cnn.param_count(), dtype=torch.float32, device=V.device)
        net.gradient(V, P, T(nbr[sel]), T(target[sel]), g)
        return g

    whole = grad(slice(0, B))
    halves = 0.5 * (grad(slice(0, B // 2)) + grad(slice(B // 2, B)))
    net.sync()
    assert float(torch.linalg.norm(whole - halves)) <= 1e-5 * float(torch.linalg.norm(halves))


def test_conv_net_sums_of_a_large_batch():
    """A float32 sum of the weight gradient takes at most 2048 pixels whatever
    the batch (4096 samples here): one sample is off by 16 and the others by
    2^-14, whose output gradients, 2^-18 of the first's, vanish in a sum that
    holds the first sample, and so must share it with three other samples at
    most.  The last bias's gradient is the sum of the output gradients, known
    exactly; the later adding of the parts is exact for these values."""
    B = 4096
    print(f"conv net sums B={B}", flush=True)
    _, vec, pats, nbr, _ = make_case(4, 40, 73)
    net, V, P = cnn.ConvInit(B), T(vec), T(pats)
    n = T(np.tile(nbr, (B // 4, 1)))
    out = net.forward(V, P, n)
    off = torch.full((B, 1, 1), 2.0 ** -14, device=out.device)
    off[0] = 16.0
    grad = torch.zeros(cnn.param_count(), dtype=torch.float32, device=out.device)
    net.gradient(V, P, n, out - off, grad)
    net.sync()
    got = cnn.unpack_params(grad.cpu().numpy())[4][1][0]
    want = 1024 * (16.0 + (B - 1) * 2.0 ** -14) * 2 / (B * 1024)
    assert abs(got - want) <= 2.0 ** -16 * want


@pytest.mark.parametrize("P,H,W", [(0, 40, 33), (1, 32, 32), (70, 100, 90)])
def test_stitch_tiles(P, H, W):
    """Patches over image edges, more than 64 of them, ragged tiles; the sum
    runs in patch order in float32 as the reference's."""
    rng = np.random.default_rng(P + H)
    patches = rng.standard_normal((P, 32, 32)).astype(np.float32)
    centres = np.stack([rng.uniform(-10, H + 10, P), rng.uniform(-10, W + 10, P)], 1).astype(np.float32)
    img = rng.standard_normal((H, W)).astype(np.float32)
    total, hits = np.zeros((H, W), np.float32), np.zeros((H, W), np.float32)
    for q in range(P):
        y0, x0 = int(np.rint(centres[q, 0])) - 16, int(np.rint(centres[q, 1])) - 16
        ya, yb, xa, xb = max(y0, 0), min(y0 + 32, H), max(x0, 0), min(x0 + 32, W)
        if ya < yb and xa < xb:
            total[ya:yb, xa:xb] += patches[q, ya - y0:yb - y0, xa - x0:xb - x0]
            hits[ya:yb, xa:xb] += 1
    ref = np.where(hits > 0, total / np.maximum(hits, 1), img)
    out = T(img)
    cnn.ConvInit(1).stitch(T(patches), T(centres), out)
    # one float division apart: at most one unit in the last place
    assert np.max(np.abs(out.cpu().numpy() - ref)) <= 2.0 ** -23 * np.max(np.abs(ref))
