"""The surrogate network on the GPU (MFMA BF16 kernels) against the FP64
network oracle, its training, and the stencil-fallback controller.

Layer by layer (test_layers_elementwise_full_path_shapes), every kernel is
compared element by element with the oracle fed the GPU's own BF16 inputs
(read back through gs_surrogate_read_tensor), under a per-element bound
|gpu - ref| <= rtol |ref| + atol derived from the kernel's arithmetic:
  - BF16 storage of a result: unit roundoff 2^-8 (rtol);
  - FP32 accumulation on the matrix cores: each v_mfma_f32_16x16x32_bf16
    adds 32 exact BF16 products to the accumulator, taken as at most 32 FP32
    roundings, so a chain of m instructions errs by at most 32 m 2^-24 S, where
    S is the same sum over absolute values (computed by the oracle);
  - the GELU kernels' erf (Abramowitz and Stegun 7.1.26 evaluated in FP32):
    at most 1e-6 absolute;
  - weight and bias gradients: per-workgroup FP32 partials (the chain is the
    workgroup's MFMAs or adds), folded in FP64, rounded once to FP32.
The shapes (2 samples of 48 x 10 x 72) cover three x-patches, a partial
y-patch, eighteen convolution z-chunks and two weight-gradient z-chunks (64
planes and a ragged 8).

End to end (forward, loss and gradients from the original inputs), the
relative L2 errors come from BF16 rounding through four layers and are
bounded by norm bars set near the measured values (forward 6-8e-3, gradients
2-3e-3)."""
import numpy as np
import pytest

from oracle import oracle as O
from oracle import surrogate_oracle as S
from synth import random_blobs, surrogate_init
from tests.gpu_util import require_gpu

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch():
    return require_gpu()


def bf16_round(x):
    x = np.asarray(x, dtype=np.float32)
    b = x.view(np.uint32).astype(np.uint64)
    b = ((b + 0x7FFF + ((b >> 16) & 1)) >> 16) << 16
    return b.astype(np.uint32).view(np.float32).astype(np.float64)


def _params(seed, last_scale=3.0):
    p = surrogate_init(seed).astype(np.float64)
    # larger last layer and nonzero biases so the correction is not tiny
    params = S.unflatten(p)
    rng = np.random.default_rng(seed + 1)
    params = [(W * (last_scale if l == 3 else 1.0), rng.normal(0, 0.05, size=b.shape)) for l, (W, b) in enumerate(params)]
    return S.flatten(params).astype(np.float32)


def _fields(shape, n, seed):
    rng = np.random.default_rng(seed)
    u = rng.uniform(0.2, 1.0, size=(n,) + shape)
    v = rng.uniform(0.0, 0.45, size=(n,) + shape)
    return u, v


@pytest.mark.parametrize("shape", [(8, 12, 16), (6, 7, 32)])
def test_forward_matches_oracle(torch, shape):
    """The forward pass against the oracle; (6, 7, 32) has two x-patches and
    an odd number of rows, so a wavefront of the two-row kernels holds a row
    past the grid. A prediction runs the hidden layers without storing their
    pre-activations: its activations equal bit for bit those of loss_grad's
    forward pass (which stores both) on the same inputs, and reading a
    pre-activation after it is refused."""
    from paper_2309_10292_amd import gs
    from paper_2309_10292_amd.surrogate import Surrogate
    n = 2
    p32 = _params(3)
    u, v = _fields(shape, n, 4)
    F, k = np.array([0.02, 0.05]), np.array([0.048, 0.062])
    nz, ny, nx = shape
    with Surrogate(nx, ny, nz, max_batch=n, params=p32) as m:
        ut = torch.from_numpy(u).cuda()
        vt = torch.from_numpy(v).cuda()
        pu, pv = m.predict(ut, vt, F, k)
        pu, pv = pu.cpu().numpy(), pv.cpu().numpy()
        # FP32 input path gives the same correction
        pu32, _ = m.predict(ut.float(), vt.float(), F, k)
        act_pred = [m.read_tensor(m.ACT, l, n) for l in range(3)]
        with pytest.raises(gs.GSError) as err:
            m.read_tensor(m.PRE, 0, n)
        assert err.value.status == gs.GS_ERR_STATE
        m.loss_grad(ut.float(), vt.float(), ut.float(), vt.float(), F, k)
        for l in range(3):
            assert np.array_equal(act_pred[l], m.read_tensor(m.ACT, l, n)), l
    params = S.unflatten(bf16_round(p32))
    # The network reads u and v as BF16 high/low pairs (about 16 significant
    # bits), so the oracle gets the fields themselves.
    for i in range(n):
        (eu, ev) = S.forward(params, u[i], v[i], float(np.float32(F[i])), float(np.float32(k[i])))
        du_e, dv_e = eu - u[i], ev - v[i]
        du_g, dv_g = pu[i] - u[i], pv[i] - v[i]
        ref = np.concatenate([du_e.ravel(), dv_e.ravel()])
        got = np.concatenate([du_g.ravel(), dv_g.ravel()])
        rel = np.linalg.norm(got - ref) / np.linalg.norm(ref)
        print(f"sample {i}: relative L2 of the correction {rel:.3e}, |ref| max {np.max(np.abs(ref)):.3e}")
        assert rel <= 1.5e-2, rel
    assert np.max(np.abs(pu32.cpu().numpy() - pu)) <= 1e-6 + 1e-2 * np.max(np.abs(pu - u))


def test_gradients_match_oracle(torch):
    from paper_2309_10292_amd.surrogate import Surrogate
    shape = (4, 8, 16)
    n = 2
    p32 = _params(7, last_scale=1.0)
    u, v = _fields(shape, n, 8)
    rng = np.random.default_rng(9)
    ut = u + 0.02 * rng.normal(size=u.shape)
    vt = v + 0.02 * rng.normal(size=v.shape)
    F, k = np.array([0.03, 0.045]), np.array([0.05, 0.06])
    with Surrogate(16, 8, 4, max_batch=n, params=p32) as m:
        T = lambda a: torch.from_numpy(a.astype(np.float32)).cuda().contiguous()
        loss, g = m.loss_grad(T(u), T(v), T(ut), T(vt), F, k, want_grad=True)
    params = S.unflatten(bf16_round(p32))
    # The GPU gets FP32 fields and reads them as BF16 high/low pairs (about 16
    # significant bits): the oracle gets the same FP32 values.
    f32 = lambda a: a.astype(np.float32).astype(np.float64)
    samples = []
    for i in range(n):
        samples.append((f32(u[i]), f32(v[i]), float(np.float32(F[i])), float(np.float32(k[i])), f32(ut[i]),
                        f32(vt[i])))
    loss_e, grads = S.loss_and_grads(params, samples)
    print(f"loss gpu {loss:.6e} oracle {loss_e:.6e}")
    assert abs(loss - loss_e) <= 2e-3 * loss_e
    ge = S.flatten(grads)
    o = 0
    for l, (W, b) in enumerate(grads):
        for arr in (W, b):
            a = g[o:o + arr.size].astype(np.float64)
            e = arr.ravel()
            o += arr.size
            rel = np.linalg.norm(a - e) / np.linalg.norm(e)
            cos = float(a @ e / (np.linalg.norm(a) * np.linalg.norm(e)))
            print(f"layer {l} {'W' if arr is W else 'b'}: rel {rel:.3e} cos {cos:.6f}")
            assert rel <= 1e-2 and cos >= 0.9999, (l, rel, cos)
    assert o == ge.size


U = 2.0 ** -24   # FP32 unit roundoff
B = 2.0 ** -8    # BF16 unit roundoff
ERF = 1e-6       # erf of the GELU kernels, absolute


def _check(name, got, ref, bound):
    err = np.abs(got - ref)
    worst = float(np.max(err / bound))
    mag = np.abs(ref)
    tight = float(np.median(bound[mag > 0] / mag[mag > 0])) if np.any(mag > 0) else float("nan")
    print(f"{name}: max |gpu - ref| {float(np.max(err)):.3e}, max |ref| {float(np.max(mag)):.3e}, "
          f"worst error / bound {worst:.3f}, median bound / |ref| {tight:.2e}")
    assert worst <= 1.0, (name, worst)


@pytest.mark.parametrize("nz, ny, nx, n", [(72, 10, 48, 2), (65, 6, 16, 1)], ids=["72x10x48x2", "65x6x16x1"])
def test_layers_elementwise_full_path_shapes(torch, nz, ny, nx, n):
    """Every layer's forward, data-gradient, weight- and bias-gradient kernel
    element by element against the oracle on the GPU's own BF16 inputs.
    The second shape ends the weight gradient's last z-chunk with a single
    plane (64 + 1) and the convolutions' with a single plane too, in one
    x-patch and a two-row last y-patch."""
    from paper_2309_10292_amd.surrogate import Surrogate
    shape = (nz, ny, nx)
    p32 = _params(13)
    u, v = _fields(shape, n, 14)
    rng = np.random.default_rng(15)
    ut = u + 0.02 * rng.normal(size=u.shape)
    vt = v + 0.02 * rng.normal(size=v.shape)
    F, k = np.array([0.025, 0.05])[:n], np.array([0.045, 0.065])[:n]
    f32 = lambda a: a.astype(np.float32).astype(np.float64)
    with Surrogate(nx, ny, nz, max_batch=n, params=p32) as m:
        T = lambda a: torch.from_numpy(a.astype(np.float32)).cuda().contiguous()
        loss, g = m.loss_grad(T(u), T(v), T(ut), T(vt), F, k, want_grad=True)
        X = m.read_tensor(m.INPUT, 0, n).astype(np.float64)
        Z = [m.read_tensor(m.PRE, l, n).astype(np.float64) for l in range(3)]
        A = [m.read_tensor(m.ACT, l, n).astype(np.float64) for l in range(3)]
        P = m.read_tensor(m.PRED, 3, n).astype(np.float64)
        D4 = m.read_tensor(m.DOUT, 3, n).astype(np.float64)
        DZ = [m.read_tensor(m.DPRE, l, n).astype(np.float64) for l in range(3)]
    params = S.unflatten(p32.astype(np.float64))
    Wb = [bf16_round(W) for W, _ in params]        # the kernels' BF16 weights
    bb = [b for _, b in params]                    # biases stay FP32
    cl = lambda a: np.moveaxis(a, -1, 0)           # (z, y, x, c) -> (c, z, y, x)
    n_terms = 2 * n * nz * ny * nx
    # chain lengths: forward / data-gradient MFMAs per output; weight-gradient
    # MFMAs per workgroup partial (work items of 16 x 4 or 16 x 8 cells by up
    # to 64 planes, at most four K chunks per wave and plane, plus the add of
    # two waves' sums where they split the chunks; the 16 x 4 items, counted
    # here, are the more numerous); bias-gradient FP32 adds per partial (at
    # most two staged chunks per lane and plane, then the fold over at most
    # 128 staging lanes)
    zc_w = 64
    items = (nx // 16) * ((ny + 3) // 4) * (-(-nz // zc_w)) * n
    per_wg = -(-items // 512)
    gam = lambda nch: 32 * nch * U
    gam_w = 32 * (per_wg * min(zc_w, nz) * 4 + 1) * U
    gam_b = (per_wg * min(zc_w, nz) * 2 + 128 + 1) * U
    gW_all = S.unflatten(g.astype(np.float64))
    sums_W = [np.zeros_like(W) for W in Wb]
    sums_b = [np.zeros_like(b) for b in bb]
    abs_W = [np.zeros_like(W) for W in Wb]
    abs_b = [np.zeros_like(b) for b in bb]
    for i in range(n):
        x = cl(X[i])
        assert np.all(x[6:] == 0.0)
        a_in = np.stack([x[0] + x[4], x[1] + x[5], x[2], x[3]])          # u, v as hi + lo pairs
        a_abs = np.stack([np.abs(x[0]) + np.abs(x[4]), np.abs(x[1]) + np.abs(x[5]), np.abs(x[2]), np.abs(x[3])])
        assert np.max(np.abs(a_in[0] - f32(u[i]))) <= 2.0 ** -15 * np.max(np.abs(u[i]))
        ins, ins_abs = [a_in], [a_abs]
        # forward, hidden layers: z = conv + b, a = GELU
        for l in range(3):
            zr = S.conv3d(ins[-1], Wb[l], bb[l])
            Sz = S.conv3d(ins_abs[-1], np.abs(Wb[l]), np.abs(bb[l]))
            gz = gam(7 if l == 0 else 27) + U
            _check(f"sample {i} layer {l} pre-activation", cl(Z[l][i]), zr, B * np.abs(zr) + (1 + B) * gz * Sz + 1e-30)
            ar = S.gelu(zr)
            _check(f"sample {i} layer {l} activation", cl(A[l][i]), ar,
                   B * np.abs(ar) + (1 + B) * (1.13 * gz * Sz + (ERF + 2 * U) * (np.abs(zr) + gz * Sz)) + 1e-30)
            ins.append(cl(A[l][i]))
            ins_abs.append(np.abs(cl(A[l][i])))
        # output layer: pred = input + conv + b in FP32
        cr = S.conv3d(ins[3], Wb[3], bb[3])
        Sc = S.conv3d(ins_abs[3], np.abs(Wb[3]), np.abs(bb[3]))
        res = np.stack([f32(u[i]), f32(v[i])])
        pr = res + cr
        _check(f"sample {i} prediction", P[:, i], pr,
               (1 + 2 * U) * gam(27) * Sc + U * np.abs(cr) * 1.01 + U * np.abs(pr) * 1.01 + 1e-30)
        # output gradient 2 (pred - target) / n_terms, stored in BF16
        d4 = cl(D4[i])
        assert np.all(d4[2:] == 0.0)
        tgt = np.stack([f32(ut[i]), f32(vt[i])])
        dr = (2.0 / n_terms) * (P[:, i] - tgt)
        _check(f"sample {i} output gradient", d4[:2], dr, (B + 4 * U) * np.abs(dr) * 1.01 + 1e-38)
        # backward: layer l's output gradient -> its weight and bias gradients,
        # and the data gradient of the layer below through GELU'
        douts = [cl(DZ[0][i]), cl(DZ[1][i]), cl(DZ[2][i]), d4[:2]]
        for l in range(3, -1, -1):
            dl = douts[l]
            sums_W[l] += S.conv3d_weight_grad(dl, ins[l])
            abs_W[l] += S.conv3d_weight_grad(np.abs(dl), ins_abs[l])
            sums_b[l] += dl.sum(axis=(1, 2, 3))
            abs_b[l] += np.abs(dl).sum(axis=(1, 2, 3))
            if l == 0:
                break
            gd = S.conv3d_input_grad(dl, Wb[l])
            Sd = S.conv3d_input_grad(np.abs(dl), np.abs(Wb[l]))
            zp = cl(Z[l - 1][i])
            gg = S.gelu_grad(zp)
            ref = gd * gg
            acc = np.abs(gd) + gam(7 if l == 3 else 27) * Sd
            _check(f"sample {i} data gradient below layer {l}", douts[l - 1], ref,
                   (B + 2 * U) * acc * (np.abs(gg) + ERF) + acc * ERF + 1.13 * gam(7 if l == 3 else 27) * Sd + 1e-38)
    for l in range(4):
        gW, gb = gW_all[l]
        _check(f"layer {l} weight gradient", gW, sums_W[l], gam_w * abs_W[l] + 2 * U * np.abs(sums_W[l]) + 1e-38)
        _check(f"layer {l} bias gradient", gb, sums_b[l], gam_b * abs_b[l] + 2 * U * np.abs(sums_b[l]) + 1e-38)
    # end to end against the oracle from the original inputs
    samples = [(f32(u[i]), f32(v[i]), float(np.float32(F[i])), float(np.float32(k[i])), f32(ut[i]), f32(vt[i]))
               for i in range(n)]
    loss_e, grads = S.loss_and_grads(S.unflatten(bf16_round(p32)), samples)
    print(f"loss gpu {loss:.6e} oracle {loss_e:.6e}")
    # the larger last layer makes the correction, and its BF16 error, large
    # against the residual: 4.2e-3 measured
    assert abs(loss - loss_e) <= 1e-2 * loss_e
    for l, (W, b) in enumerate(grads):
        for name, a, e in (("W", gW_all[l][0], W), ("b", gW_all[l][1], b)):
            rel = np.linalg.norm(a - e) / np.linalg.norm(e)
            cos = float(a.ravel() @ e.ravel() / (np.linalg.norm(a) * np.linalg.norm(e)))
            print(f"end to end layer {l} {name}: rel {rel:.3e} cos {cos:.6f}")
            assert rel <= 1e-2 and cos >= 0.9999, (l, name, rel, cos)


def test_training_reduces_loss_and_controller(torch):
    """Stencil-generated pairs (batched sweeps, random blobs) at L=32; a few
    hundred Adam steps must cut the loss; the controller keeps the stencil
    result whenever the check fails and matches the plain stencil when every
    jump is checked and rejected."""
    from paper_2309_10292_amd import gs
    from paper_2309_10292_amd.surrogate import Surrogate, generate_pairs, run_controlled, train
    L = 32
    blobs = random_blobs(8, L, seed=12, side_range=(4, 10))
    data = generate_pairs(L, blobs, steps_total=160, pair_every=32, warm=16)
    # pairs start at 16, 48, 80, 112, 144 (the last ends at step 160)
    assert data[0].shape[0] == 8 * 5
    with Surrogate(L, L, L, max_batch=4, params=surrogate_init(1)) as m:
        l0, _ = m.loss_grad(data[0][:4].contiguous(), data[1][:4].contiguous(), data[2][:4].contiguous(),
                            data[3][:4].contiguous(), data[4][:4], data[5][:4])
        hist = train(m, data, iters=150, batch=4, lr=2e-3, seed=0)
        print(f"loss {l0:.3e} -> {np.mean(hist[-10:]):.3e}")
        assert np.mean(hist[-10:]) < 0.5 * l0
        # controller: every jump checked with tol 0 -> always the stencil
        b = blobs[0]
        with gs.Sim(L, L, L, init="none", u0=np.ones((L, L, L)), v0=np.zeros((L, L, L)), F=b["F"], k=b["k"]) as s:
            s.fill_cube(b["x0"], b["y0"], b["z0"], b["side"])
            u0, v0 = s.read()
            r = run_controlled(m, s, b["F"], b["k"], jumps=3, check_every=1, tol=0.0)
            assert r["checks"] == 3 and r["fallbacks"] == 3
            u, v = s.read()
            assert s.current()[2] == 48
        ue, ve = O.run(u0, v0, 48, Du=0.2, Dv=0.1, F=b["F"], k=b["k"], dt=1.0)
        assert np.array_equal(u, ue) and np.array_equal(v, ve)
        # a failed check rolls the whole window back to its verified start and
        # recomputes it with the stencil: tol 0 with windows of 4 jumps gives
        # the plain stencil result too
        with gs.Sim(L, L, L, init="none", u0=u0, v0=v0, F=b["F"], k=b["k"]) as s:
            r = run_controlled(m, s, b["F"], b["k"], jumps=8, check_every=4, tol=0.0)
            assert r["checks"] == 2 and r["fallbacks"] == 2
            assert s.current()[2] == 128
            u, v = s.read()
        ue, ve = O.run(u0, v0, 128, Du=0.2, Dv=0.1, F=b["F"], k=b["k"], dt=1.0)
        assert np.array_equal(u, ue) and np.array_equal(v, ve)
        # with an infinite tolerance no check falls back
        with gs.Sim(L, L, L, init="none", u0=u0, v0=v0, F=b["F"], k=b["k"]) as s:
            r = run_controlled(m, s, b["F"], b["k"], jumps=8, check_every=4, tol=float("inf"))
            assert r["checks"] == 2 and r["fallbacks"] == 0 and len(r["rms"]) == 2
            assert s.current()[2] == 128
            print(f"controller rms at checks: {r['rms']}")
        # a network that produces non-finite values is always caught
        bad = m.params()
        bad[-200:] = np.float32(3e38)
        m.set_params(bad)
        with gs.Sim(L, L, L, init="none", u0=u0, v0=v0, F=b["F"], k=b["k"]) as s:
            r = run_controlled(m, s, b["F"], b["k"], jumps=4, check_every=4, tol=1.0)
            assert r["fallbacks"] == 1
            u, v = s.read()
        ue, ve = O.run(u0, v0, 64, Du=0.2, Dv=0.1, F=b["F"], k=b["k"], dt=1.0)
        assert np.array_equal(u, ue) and np.array_equal(v, ve)


def test_trained_surrogate_gain_l128(torch):
    """What the trained network gains over the stencil alone, at L=128.

    tests/data/surrogate_l128.npy holds parameters trained on the GPU by
    `python -m paper_2309_10292_amd.experiments surrogate --epochs 3 --save ...`
    (2000 stencil trajectories of random cubes at L=128, 22,500 Adam steps).
    On the experiment's four held-out trajectories (drawn after the training
    ones from the same seed, never trained on) this measures the one-jump
    error of the network and of persistence (no change over 16 steps)
    against the FP64 stencil, the controller's fallbacks with the 1e-3 check
    every 4th jump, and the time of one jump against 16 stencil steps. It
    also times the controlled run (surrogate jumps, checks, fallbacks) against
    the plain stencil over the same 128 steps: the net gain of the learned
    part at the 1e-3 tolerance. The check bounds the error of the checked jump
    only; the window's end is compared with the plain stencil as well. It
    asserts only what the measurement must show regardless of speed: over
    the four trajectories the network predicts the 16-step change clearly
    better than persistence (a quiescent trajectory alone can sit below the
    network's error floor), and the controller's result stays within its
    tolerance of the plain stencil (bitwise equal when every window falls
    back). The numbers are printed and, with GS_REPORT_DIR set, written to
    surrogate_gain_l128.json."""
    import json
    import os
    import time
    from paper_2309_10292_amd import gs
    from paper_2309_10292_amd.surrogate import JUMP, Surrogate, run_controlled
    here = os.path.dirname(os.path.abspath(__file__))
    params = np.load(os.path.join(here, "data", "surrogate_l128.npy"))
    assert params.shape == (S.N_PARAMS,) and np.all(np.isfinite(params))
    L, warm = 128, 64
    blobs = random_blobs(2004, L, seed=230910292, side_range=(6, 24))[2000:]
    report = dict(L=L, runs=[])

    def start(b, storage="f64"):
        s = gs.Sim(L, L, L, storage=storage, init="none", u0=np.ones((L,) * 3), v0=np.zeros((L,) * 3),
                   F=b["F"], k=b["k"])
        s.fill_cube(b["x0"], b["y0"], b["z0"], b["side"])
        s.step(warm)
        return s

    def rms(a, b, c, d):
        return ((gs.sqdiff(a, b) + gs.sqdiff(c, d)) / (2 * a.numel())) ** 0.5

    def timed(fn, reps):
        fn()
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        for _ in range(reps):
            fn()
        torch.cuda.synchronize()
        return (time.perf_counter() - t0) / reps * 1e3

    with Surrogate(L, L, L, max_batch=1, params=params) as m:
        for b in blobs:
            with start(b) as s:
                u, v, _ = s.current()
                u0, v0 = u.clone(), v.clone()
                pu, pv = m.predict(u0, v0, b["F"], b["k"])
                s.step(JUMP)
                u1, v1, _ = s.current()
                net, pers = rms(pu, u1, pv, v1), rms(u0, u1, v0, v1)
                ms_jump = timed(lambda: m.predict(u0, v0, b["F"], b["k"], pu, pv), 10)
                ms_stencil = timed(lambda: s.step(JUMP), 10)
            with start(b) as s, start(b) as ref:
                torch.cuda.synchronize()
                r = run_controlled(m, s, b["F"], b["k"], jumps=8, check_every=4, tol=1e-3)
                t0 = time.perf_counter()
                ref.step(8 * JUMP)
                torch.cuda.synchronize()
                stencil_s = time.perf_counter() - t0
                uc, vc, stc = s.current()
                ur, vr, str_ = ref.current()
                assert stc == str_ == warm + 8 * JUMP
                end = rms(uc, ur, vc, vr)
            run = dict(F=b["F"], k=b["k"], one_jump_rms_net=net, one_jump_rms_persistence=pers,
                       ms_surrogate_jump=ms_jump, ms_stencil_16_steps=ms_stencil, speed_gain=ms_stencil / ms_jump,
                       checks=r["checks"], fallbacks=r["fallbacks"], rms_at_checks=r["rms"], rms_end_vs_stencil=end,
                       controlled_seconds=r["seconds"], stencil_seconds=stencil_s,
                       net_gain_vs_stencil=stencil_s / r["seconds"])
            report["runs"].append(run)
            print(json.dumps(run))
            if r["fallbacks"] == r["checks"]:
                assert end == 0.0
            else:
                assert end <= 2e-3 * r["checks"], end
    net_mean = float(np.mean([x["one_jump_rms_net"] for x in report["runs"]]))
    pers_mean = float(np.mean([x["one_jump_rms_persistence"] for x in report["runs"]]))
    report.update(one_jump_rms_net_mean=net_mean, one_jump_rms_persistence_mean=pers_mean)
    print(f"one-jump RMS: network {net_mean:.3e}, persistence {pers_mean:.3e}")
    assert net_mean < 0.5 * pers_mean, (net_mean, pers_mean)
    if os.environ.get("GS_REPORT_DIR"):
        with open(os.path.join(os.environ["GS_REPORT_DIR"], "surrogate_gain_l128.json"), "w") as f:
            json.dump(report, f, indent=1)


# grids at the edges of the output layer's tiles: the narrowest, a whole row of 8 16-cell groups, one and 7 groups more
# (tiles between halo groups, the last with 1 or 3 groups), rows not a multiple of 6, a single z-plane chunk
@pytest.mark.parametrize("shape", [(4, 4, 16), (5, 8, 128), (4, 7, 144), (4, 6, 240)])
@pytest.mark.parametrize("dtype", ["float32", "float64"])
def test_output_layer_tiles(torch, shape, dtype):
    """predict()'s output layer against the FP64 layer applied to the GPU's own activations: residual plus the FP32
    accumulation of 3 MFMAs (dz), 32 roundings each, and at most 12 for the bias and the 9 shifted partial sums.
    FP32 outputs are rounded once more, and their correction is added to an FP32 residual."""
    from paper_2309_10292_amd.surrogate import Surrogate
    from synth import surrogate_init
    nz, ny, nx = shape
    rng = np.random.default_rng(sum(shape))
    p = surrogate_init(3)
    p[w_off_out():] *= 10  # the correction as large as the other layers' outputs
    u = rng.uniform(0.2, 1.0, (2,) + shape)
    v = rng.uniform(0.0, 0.5, (2,) + shape)
    with Surrogate(nx, ny, nz, max_batch=2, params=p) as m:
        tu, tv = (torch.from_numpy(a.astype(dtype)).cuda() for a in (u, v))
        ou, ov = m.predict(tu, tv, [0.02, 0.05], [0.05, 0.06])
        act = m.read_tensor(m.ACT, 2, 2).astype(np.float64)
    W = p[w_off_out():w_off_out() + 2 * 32 * 27].astype(np.float32)
    W = ((W.view(np.uint32) + 0x7FFF + ((W.view(np.uint32) >> 16) & 1)) & 0xFFFF0000).astype(np.uint32).view(np.float32)
    W = W.astype(np.float64).reshape(2, 32, 27)
    b = p[w_off_out() + 2 * 32 * 27:].astype(np.float64)
    corr = np.zeros((2,) + shape + (2,))
    mag = np.zeros_like(corr)
    for d in range(27):
        s = np.roll(act, (1 - d // 9, 1 - d // 3 % 3, 1 - d % 3), (1, 2, 3))
        corr += s @ W[:, :, d].T
        mag += np.abs(s) @ np.abs(W[:, :, d].T)
    for got, res, o in ((ou, tu, 0), (ov, tv, 1)):
        ref = res.double().cpu().numpy() + (corr[..., o] + b[o])
        bound = 2.0 ** -24 * (32 * 3 + 12) * (mag[..., o] + abs(b[o]))
        if dtype == "float32":
            bound = bound + 2.0 ** -23 * np.abs(ref)
        assert np.all(np.abs(got.double().cpu().numpy() - ref) <= bound), float(np.max(np.abs(got.double().cpu().numpy() - ref) / bound))


def w_off_out():
    """Offset of the output layer's weights in the flat parameter vector."""
    return (32 * 4 * 27 + 32) + 2 * (32 * 32 * 27 + 32)


def test_predict_more_samples_than_one_launch_packs(torch):
    """(F, k) travel with the input packing's launches, 64 samples each: 70 samples equal the samples one by one."""
    from paper_2309_10292_amd.surrogate import Surrogate
    n, shape = 70, (4, 8, 16)
    rng = np.random.default_rng(1)
    u = torch.from_numpy(rng.uniform(0.2, 1.0, (n,) + shape).astype(np.float32)).cuda()
    v = torch.from_numpy(rng.uniform(0.0, 0.5, (n,) + shape).astype(np.float32)).cuda()
    F, k = rng.uniform(0.01, 0.06, n), rng.uniform(0.04, 0.07, n)
    with Surrogate(16, 8, 4, max_batch=n) as m:
        ou, ov = m.predict(u, v, F, k)
        for i in (0, 1, 63, 64, 65, 69):
            su, sv = m.predict(u[i], v[i], F[i], k[i])
            assert torch.equal(su, ou[i]) and torch.equal(sv, ov[i]), i


# the smallest grid, and one with more work items than wavefronts at once (5000 columns of 16 x 4 cells) and rows that
# are no multiple of a patch's
@pytest.mark.parametrize("nz, ny, nx, n", [(4, 4, 16, 2), (5, 998, 320, 1)], ids=["4x4x16x2", "5x998x320x1"])
def test_edge_layer_weight_gradients(torch, nz, ny, nx, n):
    """First and last layer's weight and bias gradients against FP64 sums of the GPU's own stored tensors: FP32 sums
    of at most 32 roundings per MFMA over a wavefront's items (two K chunks per plane) and two folds, summed in FP64
    and rounded once; the last layer's bias adds lane by lane."""
    from paper_2309_10292_amd.surrogate import Surrogate
    u, v = _fields((nz, ny, nx), n, 4)
    rng = np.random.default_rng(5)
    ut, vt = u + 0.02 * rng.normal(size=u.shape), v + 0.02 * rng.normal(size=v.shape)
    F, k = np.array([0.025, 0.05])[:n], np.array([0.045, 0.065])[:n]
    T = lambda a: torch.from_numpy(a.astype(np.float32)).cuda().contiguous()
    with Surrogate(nx, ny, nz, max_batch=n, params=_params(21)) as m:
        _, g = m.loss_grad(T(u), T(v), T(ut), T(vt), F, k, want_grad=True)
        D = lambda t, l: torch.from_numpy(m.read_tensor(t, l, n)).cuda().double()
        X, A2, D0, D4 = D(m.INPUT, 0), D(m.ACT, 2), D(m.DPRE, 0), D(m.DOUT, 3)[..., :2]
    G = S.unflatten(g.astype(np.float64))
    xin = torch.stack([X[..., 0] + X[..., 4], X[..., 1] + X[..., 5], X[..., 2], X[..., 3]], -1)
    xabs = torch.stack([X[..., 0].abs() + X[..., 4].abs(), X[..., 1].abs() + X[..., 5].abs(), X[..., 2].abs(), X[..., 3].abs()], -1)
    items = -(-(nx // 16) * -(-ny // 4) * n * nz // 3072)  # items of at least one plane per wavefront, at most
    gam = (32 * 2 * (items + 2 * nz) + 4 * 64) * U
    for name, l, dz, a, a_abs in (("first", 0, D0, xin, xabs), ("last", 3, D4, A2, A2.abs())):
        co, ci = dz.shape[-1], a.shape[-1]
        for d in range(27):
            sh = (1 - d // 9, 1 - d // 3 % 3, 1 - d % 3)
            s, sa = torch.roll(a, sh, (1, 2, 3)).reshape(-1, ci), torch.roll(a_abs, sh, (1, 2, 3)).reshape(-1, ci)
            z = dz.reshape(-1, co)
            ref, mag = (z.t().contiguous() @ s).cpu().numpy(), (z.abs().t().contiguous() @ sa).cpu().numpy()
            got = G[l][0].reshape(co, ci, 27)[:, :, d]
            assert np.all(np.abs(got - ref) <= gam * mag + 2 * U * np.abs(ref) + 1e-38), (name, d)
        ref, mag = dz.reshape(-1, co).sum(0).cpu().numpy(), dz.abs().reshape(-1, co).sum(0).cpu().numpy()
        assert np.all(np.abs(G[l][1] - ref) <= gam * mag + 2 * U * np.abs(ref) + 1e-38), name


# hidden-layer launches of 12 (the second repeats planes of the first) and 16 planes per workgroup, 9 and 12 in the
# 8-channel layers, the second with an odd number of rows; the small grids' launches take 8, and 6 and 3
@pytest.mark.parametrize("nz, ny, nx, reps", [(22, 16, 64, 32), (30, 15, 128, 32)], ids=["22x16x64", "30x15x128"])
def test_hidden_layers_same_for_every_chunk(torch, nz, ny, nx, reps):
    """A grid repeated along x holds the small grid's tensors again, bit for bit (the loss gradient scaled by the
    power of two that the number of cells grew by): the planes a workgroup takes change no result."""
    from paper_2309_10292_amd.surrogate import Surrogate
    u, v = _fields((nz, ny, nx), 1, 8)
    rng = np.random.default_rng(9)
    ut, vt = u + 0.02 * rng.normal(size=u.shape), v + 0.02 * rng.normal(size=v.shape)
    got = []
    for r in (1, reps):
        T = lambda a: torch.from_numpy(np.tile(a, (1, 1, 1, r)).astype(np.float32)).cuda()
        with Surrogate(nx * r, ny, nz, params=_params(22)) as m:
            m.loss_grad(T(u), T(v), T(ut), T(vt), [0.03], [0.055], want_grad=True)
            got.append([m.read_tensor(t, l, 1)[0] for t, l in ([(t, l) for l in range(3) for t in (m.PRE, m.ACT)] + [(m.DPRE, l) for l in range(3)])])
    for i, (small, large) in enumerate(zip(*got)):
        small = small / reps if i >= 6 else small
        assert np.array_equal(large.reshape(nz, ny, reps, nx, 32), np.broadcast_to(small[:, :, None], (nz, ny, reps, nx, 32))), i


@pytest.mark.parametrize("ny", [4, 5, 9])
def test_gradients_do_not_read_other_samples(torch, ny):
    """Gradients of one sample in a workspace for two, whose unused half holds NaN: bit for bit those of a workspace
    for one. A patch of the hidden layers' weight gradients takes 10 activation rows, which wrap around the grid
    twice where it has 4."""
    from paper_2309_10292_amd.surrogate import Surrogate
    u, v = _fields((8, ny, 16), 1, 10)
    T = lambda a: torch.from_numpy(a.astype(np.float32)).cuda()
    got = []
    for batch in (1, 2):
        with Surrogate(16, ny, 8, max_batch=batch, params=_params(23)) as m:
            m.workspace.fill_(255)
            m.set_params(_params(23))
            got.append(m.loss_grad(T(u), T(v), T(u * 0.98), T(v + 0.01), [0.03], [0.055], want_grad=True))
    assert np.all(np.isfinite(got[0][1])) and got[0][0] == got[1][0] and np.array_equal(got[0][1], got[1][1])
