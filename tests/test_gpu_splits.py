"""The ways a launch is divided, at the sizes where one gives way to the next, against the FP64 oracle.

* rays: many cameras of 9x5 pixels, one workgroup each, so that every march runs with one lane per ray,
  four, eight and sixteen; wide pixels; up to eight layers; the opacity residual and jittered samples;
* a value that is not finite stays in the voxels and texels its ray touches;
* the line search, whose trials are enqueued four at a time;
* the learned preconditioner's training rows, 32 to a wave and 256 to a workgroup, and its units;
* upsampling, four voxels of a column to a thread.

Bars: those of the parity tests for the same quantities (residuals and F 1e-5; J v, J^T u, J^T J v,
gradient and blocks 1e-4, norm-wise relative): the divisions change the order of FP32 sums only.
"""
import math

import numpy as np
import pytest

import perf_synth as ps

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def rel(a, b):
    a = np.asarray(a, dtype=np.float64).reshape(-1)
    b = np.asarray(b, dtype=np.float64).reshape(-1)
    return np.linalg.norm(a - b) / max(np.linalg.norm(b), 1e-300)


def hemisphere(n, radius=2.8):
    k = np.arange(n) + 0.5
    z = 0.05 + 0.9 * k / n
    phi = math.pi * (1.0 + 5.0 ** 0.5) * k
    s = np.sqrt(1.0 - z * z)
    return radius * np.stack([s * np.cos(phi), s * np.sin(phi), z], axis=1)


RADII = tuple(2.0 + 0.5 * i for i in range(8))
# cameras of one workgroup (a 16x8 tile), field of view (14 degrees: 0.46 voxels a pixel; 60: 2.2), layers,
# opacity residual, jitter, storage
RAYS = [(899, 14.0, 1, 0.0, 0, "f32"), (900, 14.0, 8, 0.1, 3, "f32"), (1799, 14.0, 5, 0.0, 0, "bf16"),
        (1800, 14.0, 2, 0.1, 0, "f32"), (2000, 14.0, 2, 0.0, 5, "f32"), (3500, 14.0, 8, 0.1, 3, "f32"),
        (3500, 14.0, 2, 0.0, 0, "bf16"), (3500, 60.0, 3, 0.1, 0, "f32"), (40, 60.0, 8, 0.1, 3, "bf16"),
        (1, 60.0, 0, 0.0, 0, "f32"), (349, 14.0, 8, 0.1, 3, "f32"), (350, 14.0, 1, 0.0, 5, "bf16"),
        (350, 60.0, 8, 0.1, 0, "f32"), (1999, 14.0, 3, 0.1, 3, "f32")]


class Rays:
    def __init__(self, n, fov, layers, aux, jitter, dtype):
        import oracle
        from paper_2112_05598_amd.scene import Scene
        print(f"[case] {n} cameras fov={fov} layers={layers} aux={aux} jitter={jitter} {dtype}", flush=True)
        self.spec = ps.SceneSpec(12, 10, 8, layer_radii=RADII[:layers], env_w=16, env_h=9, background=(0.1, 0.2, 0.3))
        cams = ps.cameras_from_origins([tuple(o) for o in hemisphere(n)], 9, 5, fov)
        rng = np.random.default_rng(n)
        x = rng.uniform(0.0, 1.0, size=(self.spec.n_units, 4)).astype(np.float32)
        x = torch.from_numpy(x.reshape(-1))
        if dtype == "bf16":
            x = x.bfloat16().float()
        self.x64 = x.numpy().astype(np.float64)
        self.orc = oracle.OracleScene(self.spec, cams, aux_lambda=aux, jitter_seed=jitter)
        gt = np.clip(self.x64 + rng.normal(0.0, 0.2, self.x64.shape), 0.0, 1.0)
        self.targets = self.orc.render(gt)[0].astype(np.float32)
        self.sc = Scene(self.spec, cams, torch.from_numpy(self.targets.reshape(-1)).cuda(), param_dtype=dtype,
                        device="cuda:0", aux_lambda=aux)
        self.sc.set_jitter(jitter)
        self.tx = x.cuda() if dtype == "f32" else self.sc.pack_bf16(x.cuda())


@pytest.fixture(scope="module", params=RAYS, ids=lambda c: f"{c[0]}-fov{c[1]:.0f}-{c[5]}")
def rays(request):
    return Rays(*request.param)


def test_marches(rays):
    sc, orc, tx, x64 = rays.sc, rays.orc, rays.tx, rays.x64
    r, F = sc.render_residuals(tx)
    _, r_or, F_or, _ = orc.render(x64, rays.targets)
    assert rel(r.cpu().numpy(), r_or) <= 1e-5 and abs(F.item() - F_or) <= 1e-5 * F_or
    v = ps.random_vector(sc.n_params, 1)
    u = ps.random_vector(sc.n_res * sc.n_rays, 2)
    tv, tu = torch.from_numpy(v).cuda(), torch.from_numpy(u).cuda()
    assert rel(sc.apply_J(tx, tv).cpu().numpy(), orc.apply_J(x64, v.astype(np.float64))) <= 1e-4
    assert rel(sc.apply_Jt(tx, tu).cpu().numpy(), orc.apply_Jt(x64, u.astype(np.float64))) <= 1e-4
    assert rel(sc.apply_JtJ(tx, tv).cpu().numpy(), orc.apply_JtJ(x64, v.astype(np.float64))) <= 1e-4
    grad, blocks, _, F = sc.build_precond(tx, "jacobi")
    g_or, b_or, _ = orc.grad_blocks(x64, rays.targets)
    assert rel(grad.cpu().numpy(), g_or) <= 1e-4 and rel(blocks.cpu().numpy(), b_or) <= 1e-4
    assert abs(F.item() - F_or) <= 1e-5 * F_or


@pytest.mark.parametrize("n", [30, 1000, 2000, 3500])
def test_nonfinite_stays_in_its_corners(n):
    s = Rays(n, 14.0, 2, 0.0, 0, "f32")
    u = ps.random_vector(3 * s.sc.n_rays, 4)
    ray = 45 * (n // 2) + 22  # the middle of an image
    u[3 * ray:3 * ray + 3] = 0.0
    y_or = s.orc.apply_Jt(s.x64, u.astype(np.float64)).reshape(-1, 4)
    u[3 * ray] = np.inf
    y = s.sc.apply_Jt(s.tx, torch.from_numpy(u).cuda()).cpu().numpy().reshape(-1, 4)
    unit = np.unique(s.orc.ray_row(s.x64, ray)[0])
    # a sample's corners of weight zero (it lies on a face of its cell, or was clamped to the grid) are not in
    # the oracle's row, but 0 * inf is added to them: each shares a cell with a corner that is
    z, y_, x = np.unravel_index(unit[unit < s.spec.n_vox], (8, 10, 12))
    near = np.zeros((10, 12, 14), bool)
    for k in np.ndindex(3, 3, 3):
        near[z + k[0], y_ + k[1], x + k[2]] = True
    touched = np.concatenate([np.flatnonzero(near[1:-1, 1:-1, 1:-1]), unit[unit >= s.spec.n_vox]])
    others = np.setdiff1d(np.arange(s.spec.n_units), touched)
    assert not np.isfinite(y[touched]).all() and np.isfinite(y[others]).all()
    assert rel(y[others], y_or[others]) <= 1e-4


@pytest.mark.parametrize("ls_max", [1, 3, 4, 5, 8, 9, 20])
def test_line_search_batches(ls_max):
    """The trials of a batch behind the one that ends the search count for nothing."""
    import oracle
    from paper_2112_05598_amd.scene import Scene
    w = ps.workload("small")
    orc = oracle.OracleScene(w.spec, w.cams)
    targets = orc.render(w.x_gt)[0].astype(np.float32)
    sc = Scene(w.spec, w.cams, torch.from_numpy(targets.reshape(-1)).cuda(), device="cuda:0")
    x = torch.from_numpy(w.x_init.astype(np.float32)).cuda()
    st = sc.gn_step(x, max_iters=4, ls_max=ls_max)
    ref = oracle.gn_step(orc, w.x_init.astype(np.float64), targets, max_iters=4, ls_max=ls_max)
    print(f"[case] ls_max={ls_max}: {ref['n_ls']} trials, gamma {ref['gamma']}", flush=True)
    assert st["ls_trials"] == ref["n_ls"]
    assert abs(st["gamma"] - ref["gamma"]) <= 1e-6
    assert abs(st["F_after"] - ref["F_after"]) <= 1e-3 * ref["F_before"]
    # the parameters are those of the accepted step
    assert abs(float(sc.render_residuals(x)[1]) - st["F_after"]) <= 1e-5 * st["F_before"]


def unit_rows(n, seed):
    from oracle import mlp
    rng = np.random.default_rng(seed)
    d, f = 10.0 ** rng.uniform(-2, 1, n), 10.0 ** rng.uniform(-2, 1, n)
    e = rng.uniform(-0.5, 0.5, (n, 3)) * np.sqrt(d * f)[:, None]
    blocks = np.concatenate([d[:, None], e, f[:, None]], axis=1).astype(np.float32)
    feat = mlp.features(rng.uniform(0.0, 1.0, 4 * n), blocks.astype(np.float64)).astype(np.float32)
    return feat, blocks


@pytest.mark.parametrize("n,shift", [(1, 0), (31, 0), (32, 0), (33, 1), (255, 0), (257, 0), (32769, 0)])
def test_training_rows(n, shift):
    """Bars of the training-gradient test; `shift` elements off the allocations' alignment."""
    from oracle import mlp
    from paper_2112_05598_amd.scene import mlp_train_step
    print(f"[case] {n} rows, shift {shift}", flush=True)
    feat, blocks = unit_rows(n, n)
    rng = np.random.default_rng(1)
    p = mlp.unpack(mlp.init_weights(5) + 0.05 * rng.normal(size=mlp.NW))
    p["W1"][:, mlp.N_NET:] = 0
    p["W3"][10:] = 0
    bits = mlp.bf16_bits(mlp.pack(p))
    wq = mlp.bits_to_f64(bits)

    def at(a):
        t = torch.zeros(a.size + shift, dtype=torch.from_numpy(a[:0]).dtype, device="cuda")[shift:]
        t.copy_(torch.from_numpy(a.reshape(-1)))
        return t
    w32, wbf = at(wq.astype(np.float32)), at(bits.view(np.int16)).view(torch.bfloat16)
    m, v, g = (at(np.zeros(mlp.NW, np.float32)) for _ in range(3))
    loss = torch.zeros(1, device="cuda")
    n64 = mlp.feature_stats(unit_rows(4096, 0)[0].astype(np.float64))
    norm = torch.from_numpy(n64.astype(np.float32)).cuda()
    mlp_train_step(w32, wbf, m, v, 1, 1e-4, norm, torch.from_numpy(feat).cuda(), torch.from_numpy(blocks).cuda(), loss, g)
    L_or, g_or = mlp.loss_and_grad(wq, n64, feat.astype(np.float64), blocks.astype(np.float64))
    grad = (m / 0.1).cpu().numpy()
    assert abs(loss.item() - L_or) <= 2e-2 * L_or
    assert rel(grad, g_or) <= 5e-2
    # the second copy of the weights is the first one's rounding
    assert torch.equal(wbf, w32.to(torch.bfloat16))


@pytest.mark.parametrize("src,dst", [((2, 2, 2), (3, 5, 7)), ((5, 3, 4), (9, 6, 8)), ((6, 7, 5), (13, 14, 9)),
                                     ((4, 4, 9), (4, 5, 17))])
def test_upsampling_columns(src, dst):
    import oracle
    from paper_2112_05598_amd.scene import upsample
    sf, st = (ps.SceneSpec(*s, layer_radii=(2.0, 3.0), env_w=w, env_h=h) for s, w, h in ((src, 7, 5), (dst, 13, 9)))
    print(f"[case] upsample {src} -> {dst}", flush=True)
    x = np.random.default_rng(3).uniform(0.0, 1.0, 4 * sf.n_units).astype(np.float32)
    y = upsample(sf, torch.from_numpy(x).cuda(), st).cpu().numpy()
    np.testing.assert_allclose(y, oracle.upsample(sf, x.astype(np.float64), st), rtol=1e-6, atol=1e-6)
