"""Squaring kernels at the edges of their tiles: the direct-to-LDS 64-tile split kernel, the
FP64 kernel on mixed 64 / 32 tiles, the fragment-major split kernels, and the control of a
layer run by a squaring launch, each against the kernel that computes the same chain of
products (bit for bit) or exact FP64 arithmetic."""
import numpy as np
import pytest
import torch

from paper_2101_06385_amd import sp2, workloads as wl

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def _sym(n, seed, dtype):
    x = np.random.default_rng(seed).standard_normal((n, n)) / np.sqrt(n)
    return torch.from_numpy(0.5 * (x + x.T)).to(DEV, dtype)


@pytest.mark.parametrize("prec", ["fp16x2", "bf16x2"])
@pytest.mark.parametrize("n", [1, 31, 64, 65, 127, 200, 833])
def test_split_64_tile_pipeline_equals_register_staged_kernel(prec, n):
    x = _sym(n, 500 + n, torch.float32)
    for coef in ((1.0, 0.0, 0.0), (-1.0, 2.0, 0.25)):
        y, s = sp2.square(x, *coef, precision=prec, tile=64, kernel=1)
        y8, s8 = sp2.square(x, *coef, precision=prec, tile=64, kernel=8)
        assert torch.equal(y, y8) and s == s8


# 1472: 276 64-tiles = 256 whole + 20 cut; 1408: 253, all cut
@pytest.mark.parametrize("n", [1, 15, 16, 17, 33, 63, 65, 129, 700, 1400, 1472])
def test_fp64_mixed_tiles_equal_128_tiles_and_exact_square(n):
    x = _sym(n, 600 + n, torch.float64)
    alpha, beta, gamma = -1.0, 2.0, 0.5
    y, s = sp2.square(x, alpha, beta, gamma, precision="fp64", tile=128, kernel=0)
    y4, _ = sp2.square(x, alpha, beta, gamma, precision="fp64", tile=128, kernel=4)
    assert torch.equal(y, y4) and torch.equal(y, y.T)
    xc = x.cpu().numpy()
    ref = alpha * (xc @ xc) + beta * xc + gamma * np.eye(n)
    # each side: n products and sums, then three more operations
    bound = 2 * (n + 3) * 2.0**-53 * (np.abs(xc) @ np.abs(xc) + 2 * np.abs(xc) + np.abs(gamma) * np.eye(n))
    assert np.all(np.abs(y.cpu().numpy() - ref) <= bound + 1e-300)
    got = y.cpu().numpy()
    terms = n * n + 1   # additions of the sum of squares in any order
    assert abs(s[0] - np.trace(got)) <= 2 * n * 2.0**-53 * np.abs(np.diag(got)).sum()
    assert abs(s[1] - (got**2).sum()) <= 2 * terms * 2.0**-53 * (got**2).sum()


@pytest.mark.parametrize("prec", ["fp16x2", "bf16x2"])
@pytest.mark.parametrize("n,gap", [(10, None), (64, None), (300, None), (777, (-0.9, 0.9))])
def test_control_in_the_squaring_launch_equals_separate_control(prec, n, gap):
    """tile 64: kernel 1 runs the control in the squaring launches, kernel 8 has control
    launches; the histories and D are the same bits."""
    w = wl.gapped(700 + n, n, n // 2)
    h = torch.from_numpy(w.h).to(DEV)
    d, i = sp2.density(h, w.n_occ, precision=prec, tile=64, kernel=1, gap=gap)
    d8, i8 = sp2.density(h, w.n_occ, precision=prec, tile=64, kernel=8, gap=gap)
    assert torch.equal(d, d8)
    for k in ("status", "layers", "sigma", "iderr", "ns", "nx", "sigma_c", "accelerated", "trace"):
        assert i[k] == i8[k], k
    d2, i2 = sp2.density(h, w.n_occ, precision=prec, tile=64, kernel=1, gap=gap, max_layers=7)
    d28, i28 = sp2.density(h, w.n_occ, precision=prec, tile=64, kernel=8, gap=gap, max_layers=7)
    assert torch.equal(d2, d28) and i2["layers"] == i28["layers"] == 7 and i2["status"] == i28["status"]


# fragment-major kernels: 32-blocks and 16-wide units of K that are partly or wholly padding; 4-wave
# workgroups up to 512 64-tiles (n = 1984), one wave per tile above
@pytest.mark.parametrize("prec,n", [("fp16x2", 2), ("bf16x2", 15), ("fp16x2", 17), ("fp16x2", 33), ("bf16x2", 48),
                                    ("fp16x2", 96), ("bf16x2", 97), ("fp16x2", 129), ("fp16x2", 449),
                                    ("fp16x2", 1984), ("bf16x2", 1985), ("fp16x2", 2040)])
def test_fragment_major_layers_equal_register_staged_layers(prec, n):
    w = wl.gapped(800 + n, n, max(1, n // 2), device=DEV if n > 1000 else None)
    h = torch.from_numpy(w.h).to(DEV)
    for kw in (dict(), dict(refine=False), dict(max_layers=3, refine=False)):
        d, i = sp2.density(h, w.n_occ, precision=prec, tile=64, kernel=1, **kw)
        d8, i8 = sp2.density(h, w.n_occ, precision=prec, tile=64, kernel=8, **kw)
        assert torch.equal(d, d8) and torch.equal(d, d.T.contiguous())
        for k in ("status", "layers", "sigma", "iderr", "ns", "nx"):
            assert i[k] == i8[k], k


@pytest.mark.parametrize("n", [130, 2050, 2943])
def test_fragment_major_128_tile_order_equals_grouped_kernel(n):
    """tile 128: the grouped kernel keeps row-major planes and 128-tiles."""
    w = wl.gapped(900 + n, n, n // 3, device=DEV if n > 1000 else None)
    h = torch.from_numpy(w.h).to(DEV)
    d, i = sp2.density(h, w.n_occ, tile=128, kernel=1)
    (dg,), (ig,) = sp2.density_batched([h], [w.n_occ], tile=128)
    assert torch.equal(d, dg)
    assert i["sigma"] == ig["sigma"] and i["status"] == ig["status"] == sp2.SP2_OK


def test_fragment_major_async_call_and_layer_cap():
    """Asynchronous calls enqueue every layer: the ones behind the stop return at once, with the
    state carried through both hot blocks (odd and even caps)."""
    w = wl.gapped(950, 500, 200)
    h = torch.from_numpy(w.h).to(DEV)
    d, i = sp2.density(h, w.n_occ)
    for cap in (100, 101):
        ws = sp2.alloc_workspace(sp2.workspace_size(500, sp2.options(max_layers=cap)), DEV)
        da, _ = sp2.density(h, w.n_occ, sync=False, max_layers=cap, workspace=ws)
        torch.cuda.synchronize()
        q = sp2.query(ws, 500, max_layers=cap)
        assert torch.equal(da, d)
        for k in ("status", "layers", "sigma", "iderr", "trace", "converged"):
            assert q[k] == i[k], k


# one workgroup per solve up to n = 64: one and two 32-blocks, ragged 16-wide units of K
@pytest.mark.parametrize("prec", ["fp16x2", "bf16x2", "fp64"])
@pytest.mark.parametrize("n", [2, 3, 15, 16, 17, 32, 33, 50, 64])
def test_one_workgroup_solve_equals_layer_launches(prec, n):
    w = wl.gapped(1000 + n, n, max(1, n // 2))
    big = torch.zeros((n, n + 7), dtype=torch.float64, device=DEV)
    big[:, :n] = torch.from_numpy(w.h)
    h = big[:, :n]
    for kw in (dict(), dict(refine=False), dict(gap=(-0.9, 0.8), want_energy=True), dict(max_layers=4),
               dict(bounds=(-21.0, 22.0))):
        out = torch.full((n, n + 3), 9.0, dtype=torch.float64, device=DEV)
        d, i = sp2.density(h, w.n_occ, precision=prec, out=out[:, :n], **kw)
        d1, i1 = sp2.density(h, w.n_occ, precision=prec, tile=64, kernel=5 if prec == "fp64" else 1, **kw)
        assert torch.equal(d, d1) and torch.all(out[:, n:] == 9.0)
        for k in ("status", "layers", "converged", "sigma", "accelerated", "gap_violation", "emin", "emax", "asym"):
            assert i[k] == i1[k], (k, kw)
        # sums of n^2 terms in another order
        for k in ("trace", "energy"):
            scale = float((d.abs() * (h.abs() if k == "energy" else 1.0)).sum())
            assert abs(i[k] - i1[k]) <= 2 * (n * n + 1) * 2.0**-53 * scale, k


def test_one_workgroup_solve_reports_bad_input():
    w = wl.gapped(1100, 20, 8)
    for change, name in ((float("nan"), "ENONFINITE"), (w.h[3, 4] + 1e-3, "EINVAL")):
        x = w.h.copy()
        x[3, 4] = change
        _, i = sp2.density(torch.from_numpy(x).to(DEV), w.n_occ)
        _, i1 = sp2.density(torch.from_numpy(x).to(DEV), w.n_occ, tile=64, kernel=1)
        assert i["status_name"] == i1["status_name"] == name


# FP64 layers with the control at their head (every 64-tile cut: n <= 1408, stages in rows of 256 bytes
# up to 960) and in their last tile
@pytest.mark.parametrize("n", [65, 100, 257, 960, 961, 1408, 1409])
def test_fp64_layers_equal_128_tile_layers(n):
    w = wl.gapped(1200 + n, n, n // 2, device=DEV if n > 1000 else None)
    h = torch.from_numpy(w.h).to(DEV)
    for kw in (dict(refine=False, max_layers=3), dict(max_layers=6), dict(gap=(-0.9, 0.9), max_layers=5, refine=False)):
        d, i = sp2.density(h, w.n_occ, precision="fp64", tile=128, **kw)
        d4, i4 = sp2.density(h, w.n_occ, precision="fp64", tile=128, kernel=4, **kw)   # separate arrivals, 128-tiles
        assert torch.equal(d, d4) and i["sigma"] == i4["sigma"] and i["layers"] == i4["layers"]
        for a, b in zip(i["ns"] + i["nx"], i4["ns"] + i4["nx"]):
            assert abs(a - b) <= 2 * (n * n + 1) * 2.0**-53 * n   # sums of n^2 terms of a matrix with norm <= sqrt(n)


# FP32 layers: with the control at their head (n <= 1408; stages in rows of 256 bytes up to 960) or in
# their last tile (1409, 1472: whole 64-tiles and cut ones) against the register-staged kernel with
# control launches
@pytest.mark.parametrize("n", [65, 100, 257, 960, 961, 1408, 1409, 1472])
def test_fp32_layers_equal_register_staged_layers(n):
    w = wl.gapped(1300 + n, n, n // 2, device=DEV if n > 1000 else None)
    h = torch.from_numpy(w.h).to(DEV)
    for kw in (dict(max_layers=3), dict(max_layers=6), dict(gap=(-0.9, 0.9), max_layers=5)):
        d, i = sp2.density(h, w.n_occ, precision="fp32", refine=False, **kw)
        d1, i1 = sp2.density(h, w.n_occ, precision="fp32", refine=False, kernel=1, **kw)
        assert torch.equal(d, d1) and i["sigma"] == i1["sigma"] and i["layers"] == i1["layers"]
        for a, b in zip(i["ns"] + i["nx"], i1["ns"] + i1["nx"]):
            assert abs(a - b) <= 2 * (n * n + 1) * 2.0**-53 * n   # sums of n^2 terms of a matrix with norm <= sqrt(n)


@pytest.mark.parametrize("n", [1, 31, 33, 65, 129, 700, 1472])
def test_fp32_mixed_tiles_equal_register_staged_kernel(n):
    x = _sym(n, 1400 + n, torch.float32)
    y, s = sp2.square(x, -1.0, 2.0, 0.5, precision="fp32")
    y1, s1 = sp2.square(x, -1.0, 2.0, 0.5, precision="fp32", kernel=1)
    assert torch.equal(y, y1) and torch.equal(y, y.T)
    assert abs(s[1] - s1[1]) <= 2 * (n * n + 1) * 2.0**-53 * s1[1]
    buf = torch.empty(n * n + 1, device=DEV)   # rows that are not 16-byte aligned
    z = torch.as_strided(buf, (n, n), (n, 1), 1).copy_(x)
    assert torch.equal(sp2.square(z, -1.0, 2.0, 0.5, precision="fp32")[0], y)


def test_fp32_batch_equals_single_calls():
    ns = (5, 64, 65, 130, 300, 1472)
    ws = [wl.gapped(1500 + n, n, n // 2, device=DEV if n > 1000 else None) for n in ns]
    hs = [torch.from_numpy(w.h).to(DEV) for w in ws]
    ds, infos = sp2.density_batched(hs, [w.n_occ for w in ws], precision="fp32")
    for h, w, d, i in zip(hs, ws, ds, infos):
        d1, i1 = sp2.density(h, w.n_occ, precision="fp32", kernel=1)
        assert torch.equal(d, d1) and i["sigma"] == i1["sigma"]


# the read-out takes up to six (FP64: four) layer outputs per pass
@pytest.mark.parametrize("prec", ["fp64", "fp32", "fp16x2", "bf16x2"])
@pytest.mark.parametrize("layers", [1, 3, 4, 5, 6, 7, 11, 12])
def test_fermi_read_out_over_several_passes(prec, layers):
    n = 131
    h = _sym(n, 1600 + layers, torch.float64)
    rng = np.random.default_rng(layers)
    theta = np.array([(1.0, 0.0, 0.0) if b else (-1.0, 2.0, 0.0) for b in rng.integers(0, 2, layers)])
    c = rng.standard_normal(layers + 1)
    eye = np.eye(n)
    xs = []   # X_k = I - D for the read-out of X_k alone
    for k in range(layers + 1):
        d, _ = sp2.fermi_apply(h, theta, np.eye(layers + 1)[k], (-3.0, 3.0), precision=prec)
        xs.append(eye - d.cpu().numpy())
    buf = torch.empty(n, n + 5, dtype=torch.float64, device=DEV)
    d, obs = sp2.fermi_apply(h, theta, c, (-3.0, 3.0), precision=prec, out=buf[:, 1:n + 1])
    d = d.cpu().numpy()
    ref = eye - sum(ck * x for ck, x in zip(c, xs))
    scale = 1.0 + sum(abs(ck) * (1.0 + np.abs(x).max()) for ck, x in zip(c, xs))
    assert np.abs(d - ref).max() <= 2 * (layers + 4) * 2.0**-53 * scale
    hn, slack = h.cpu().numpy(), 2 * (n * n + 1) * 2.0**-53
    assert abs(obs[0] - np.trace(d)) <= slack * np.abs(np.diag(d)).sum()
    assert abs(obs[1] - (d * d).sum()) <= slack * (d * d).sum()
    assert abs(obs[2] - (d * hn).sum()) <= slack * np.abs(d * hn).sum()


# adjoint tiles: one ragged tile, several cut ones, and whole 64-tiles with cut ones (1409)
@pytest.mark.parametrize("n,layers", [(1, 1), (31, 2), (33, 3), (65, 4), (200, 5), (1409, 2)])
def test_adjoint_tiles_match_fp64(n, layers):
    x0, gk = _sym(n, 1700 + n, torch.float32), _sym(n, 1800 + n, torch.float32)
    rng = np.random.default_rng(n)
    w, b, c = (torch.from_numpy(rng.uniform(0.2, 0.8, layers).astype(np.float32)).to(DEV) for _ in range(3))
    xk, ws = sp2.net_forward(x0, w, b, c, precision="fp32")
    dw, db, dc, g0 = sp2.net_backward(gk, w, b, c, ws, precision="fp32")
    xs = [x0.double().cpu().numpy()]
    eye = np.eye(n)
    wd, bd, cd = (v.double().cpu().numpy() for v in (w, b, c))
    for k in range(layers):
        xs.append(wd[k] * xs[-1] @ xs[-1] + bd[k] * xs[-1] + cd[k] * eye)
    g = gk.double().cpu().numpy()
    u = 2.0**-24
    # Forward and adjoint layers are each 2 n + 4 roundings of at most |W| |X| |X| + |B| |X| + |c| in
    # norm; the errors of X_k enter the adjoint once more per layer.  Frobenius norms, layer by layer.
    nrm = np.linalg.norm
    ex = [0.0]
    for k in range(layers):
        a = nrm(xs[k])
        ex.append((2 * wd[k] * a + bd[k]) * ex[-1] + (2 * n + 4) * u * (wd[k] * a * a + bd[k] * a + cd[k] * n**0.5))
    eg = 0.0
    for k in range(layers - 1, -1, -1):
        x, a, gn = xs[k], nrm(xs[k]), nrm(g)
        for got, ref, m in ((dc[k], np.trace(g), n**0.5), (db[k], (g * x).sum(), a), (dw[k], (g * (x @ x)).sum(), a * a)):
            err = eg * m + gn * (2 * ex[k] * max(a, 1.0) + (2 * n + 8) * u * m)
            assert abs(float(got) - ref) <= err, (k, float(got), ref, err)
        eg = (2 * wd[k] * a + bd[k]) * eg + gn * (2 * wd[k] * ex[k] + (2 * n + 8) * u * (2 * wd[k] * a + bd[k]))
        g = wd[k] * (g @ x + x @ g) + bd[k] * g
    g0 = g0.double().cpu().numpy()
    assert np.array_equal(g0, g0.T) and nrm(g0 - g) <= eg


# network layers on fragment-major planes: 4-wave workgroups, one wave per tile (2050), blocks of a
# 64-tile beyond the data (65, 200), 64- and 128-tile product order (from 257)
@pytest.mark.parametrize("prec", ["fp16x2", "bf16x2"])
@pytest.mark.parametrize("n", [1, 16, 33, 65, 200, 256, 257, 700, 2050])
def test_fragment_major_network_layers_equal_per_tile_layers(prec, n):
    x0 = _sym(n, 1900 + n, torch.float32)
    w, b, c = (torch.tensor(v, device=DEV) for v in ([1.0, -0.5, 0.7], [0.0, 1.5, -0.25], [0.0, 0.25, -0.5]))
    for ckpt in (0, 2):
        need = sp2.net_workspace_size(n, 3, prec, ckpt)
        ws = sp2.alloc_workspace(need, DEV).fill_(255)   # NaN wherever a kernel reads what none has written
        xk, ws = sp2.net_forward(x0, w, b, c, precision=prec, ckpt_every=ckpt, workspace=ws)
        x, tile = x0, 64 if n <= 256 else 128
        for k in range(3):
            x, _ = sp2.square(x, float(w[k]), float(b[k]), float(c[k]), precision=prec, tile=tile, kernel=1)
        assert torch.equal(xk, x)
        dw, db, dc, g0 = sp2.net_backward(x0, w, b, c, ws, precision=prec, ckpt_every=ckpt)
        assert all(bool(torch.isfinite(t).all()) for t in (dw, db, dc, g0))
        if ckpt == 0:
            first = (dw, db, dc, g0)
        else:   # recomputed layers have the forward's bits
            assert all(torch.equal(p, q) for p, q in zip(first, (dw, db, dc, g0)))


@pytest.mark.parametrize("prec", ["fp16x2", "bf16x2"])
@pytest.mark.parametrize("n", [1, 33, 65, 131, 700, 2050])
def test_fragment_major_fermi_layers_equal_register_staged_layers(prec, n):
    h = _sym(n, 2000 + n, torch.float64)
    theta = np.array([(0.9, 0.0, 0.1), (-1.0, 2.0, 0.0), (1.0, -0.5, 0.25)])
    c = [0.5, -0.25, 0.125, 0.75]
    need = sp2.fermi_workspace_size(n, (-3.0, 3.0), prec, tile=64)
    ws = sp2.alloc_workspace(need, DEV).fill_(255)   # NaN wherever a kernel reads what none has written
    d, obs = sp2.fermi_apply(h, theta, c, (-3.0, 3.0), precision=prec, tile=64, workspace=ws)
    d8, obs8 = sp2.fermi_apply(h, theta, c, (-3.0, 3.0), precision=prec, tile=64, kernel=8)
    assert torch.equal(d, d8) and obs == obs8


# batches whose largest problem has n < 1024 run the 64-tile pipeline with four stages: one to
# four units of K behind the prologue, whole and ragged tiles, problems that stop at different layers
@pytest.mark.parametrize("prec", ["fp16x2", "bf16x2"])
def test_split_batch_on_64_tiles_equals_register_staged_single_calls(prec):
    ns = (2, 33, 64, 65, 128, 200, 257, 640, 1000)
    ws = [wl.gapped(2100 + n, n, max(1, n // 2)) for n in ns]
    hs = [torch.from_numpy(w.h).to(DEV) for w in ws]
    ds, infos = sp2.density_batched(hs, [w.n_occ for w in ws], precision=prec)
    for h, w, d, i in zip(hs, ws, ds, infos):
        d1, i1 = sp2.density(h, w.n_occ, precision=prec, tile=64, kernel=8)
        assert torch.equal(d, d1)
        assert i["sigma"] == i1["sigma"] and i["layers"] == i1["layers"] and i["status"] == i1["status"] == sp2.SP2_OK


# n <= 64: a timed call runs the one-workgroup solve that an untimed one runs
@pytest.mark.parametrize("prec", ["fp16x2", "bf16x2", "fp64"])
@pytest.mark.parametrize("n", [2, 10, 33, 64])
def test_timed_call_of_one_workgroup_solve_is_the_untimed_one(prec, n):
    w = wl.gapped(2200 + n, n, max(1, n // 2))
    h = torch.from_numpy(w.h).to(DEV)
    for kw in (dict(), dict(refine=False), dict(gap=(-0.9, 0.8)), dict(max_layers=4)):
        d, i = sp2.density(h, w.n_occ, precision=prec, want_energy=True, **kw)
        for _ in range(2):
            dt, it, tm = sp2.density(h, w.n_occ, precision=prec, want_energy=True, timed=True, **kw)
            assert torch.equal(d, dt) and it == i
            ran = tm["squarings"]
            assert ran == i["layers"] - (1 if i["converged"] else 0)
            assert all(x > 0 for x in tm["square_ms"][:ran]) and not any(tm["square_ms"][ran:])
            phases = tm["prep_ms"], tm["loop_ms"], tm["refine_ms"], tm["final_ms"]
            assert min(phases[0], phases[1], phases[3]) > 0 and phases[2] >= 0
            # ticks of 1e-5 ms; the event in front of the launch and the one behind it enclose it
            assert sum(phases) <= tm["total_ms"]
            assert sum(tm["square_ms"]) <= tm["loop_active_ms"] + 1e-5 * (ran + 1) <= tm["loop_ms"] + 2e-5 * (ran + 1)
            assert (min(tm["refine_square_ms"]) > 0) == (kw.get("refine") is not False)


# one layer on 64-tiles with the schedule left open: more than two, at most three tiles per CU (513 .. 768)
# take the register-staged kernel; 496, 528, 741 and 780 tiles
@pytest.mark.parametrize("prec", ["fp16x2", "bf16x2"])
@pytest.mark.parametrize("n", [1984, 1985, 2432, 2433])
def test_split_layer_of_either_schedule_has_the_same_bits(prec, n):
    x = _sym(n, 2300 + n, torch.float32)
    y, s = sp2.square(x, -1.0, 2.0, 0.25, precision=prec, tile=64)
    y1, s1 = sp2.square(x, -1.0, 2.0, 0.25, precision=prec, tile=64, kernel=1)
    assert torch.equal(y, y1) and s == s1
