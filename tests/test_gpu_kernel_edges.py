"""Kernels at the sizes where their tiles, parts and dispatch rules change,
against the FP64 oracle."""
import dataclasses

import numpy as np
import pytest

import workloads as W
from oracle import covariance as ocov
from oracle import field as ofield
from oracle import step as ostep
from parity import check_mag, params_for, split_grads

pytestmark = pytest.mark.gpu


def _t(torch, dev, a):
    return torch.from_numpy(np.ascontiguousarray(a)).to(dev)


# sixteen levels that each fit one bin of 8192 entries (the largest a level may have)
SMALL_TABLES = dataclasses.replace(W.C2_FIELD, log2_table=13, max_res=256)


@pytest.mark.parametrize("spec,S", [(W.C1_FIELD, 64), (W.C1_FIELD, 226), (W.C1_FIELD, 1023), (W.C1_FIELD, 1025),
                                    (W.C1_FIELD, 131073), (SMALL_TABLES, 16), (SMALL_TABLES, 3001)],
                         ids=["sorted", "one-part", "one-used", "two-used", "all-parts", "16-sorted", "16-levels"])
def test_scatter_of_single_bin_levels(nsl, gpu, spec, S):
    """nsl_encode_bwd where every level fits one bin: too few samples for a
    part (the counting sort), one part, parts of unequal size, every part;
    overwriting and accumulating, at 1e-5 (FP32 values) and 2e-2 (BF16)."""
    import torch
    f = nsl.Field(spec)
    nt = f.layout["table_floats"]
    rng = np.random.default_rng(S)
    xn = rng.uniform(size=(S, 3)).astype(np.float32)
    xn[: S // 2] = np.clip(0.4 + 1e-3 * np.arange(S // 2)[:, None] / max(1, S // 2), 0, 1)    # runs in shared cells
    de = rng.normal(size=(spec.levels, S, 2)).astype(np.float32)
    _, _, corners = ofield.encode_fwd(spec, np.zeros(nt), xn)
    de_sf = de.transpose(1, 0, 2).reshape(S, 2 * spec.levels).astype(np.float64)
    gt, gtm = ofield.encode_bwd(spec, corners, de_sf, np.abs(de_sf), nt)
    X, DE = _t(torch, gpu, xn), _t(torch, gpu, de)
    for prec, tol in ((nsl.PRECISION_FP32, 1e-5), (nsl.PRECISION_MIXED, 2e-2)):
        for overwrite, before in ((True, 0.0), (False, 0.5)):
            G = torch.full((f.layout["total"],), 0.5, device=gpu)
            nsl.encode_bwd(f, X, DE, G, precision=prec, overwrite=overwrite)
            g = G.cpu().numpy().astype(np.float64)
            check_mag(f"single-bin scatter p{prec}", g[:nt], gt + before, gtm + before, tol)
            assert np.all(g[nt:] == 0.5)
            assert np.all(g[:nt][gtm == 0] == before)


@pytest.mark.parametrize("spec", [W.C1_FIELD, W.C2_FIELD], ids=["tiny", "full"])
@pytest.mark.parametrize("S", [1, 16, 17, 113, 128, 129, 32768, 32897, 65553])
def test_mlp_backward_at_step_edges(nsl, gpu, spec, S):
    """nsl_mlp_bwd around its tiles of 16 samples, steps of 128 and rounds of
    256 workgroups: dL/de and the weight gradients at 1e-5 of their magnitudes,
    as the entry-point test."""
    import torch
    f = nsl.Field(spec)
    L = spec.levels
    flat, _, w64 = params_for(spec, f.layout, seed=6, table_range=0.5)
    rng = np.random.default_rng(S)
    e = rng.normal(scale=0.3, size=(S, 2 * L)).astype(np.float32)
    d = rng.normal(size=(S, 3))
    d = (d / np.linalg.norm(d, axis=1, keepdims=True)).astype(np.float32)
    dsig = rng.normal(size=S).astype(np.float32)
    drgb = rng.normal(size=(S, 3)).astype(np.float32)
    ws = torch.empty(f.workspace_bytes(S), dtype=torch.uint8, device=gpu)
    G = torch.full((f.layout["total"],), 0.5, device=gpu)
    de = nsl.mlp_bwd(f, _t(torch, gpu, flat), _t(torch, gpu, e.reshape(S, L, 2).transpose(1, 0, 2)), _t(torch, gpu, d),
                     _t(torch, gpu, dsig), _t(torch, gpu, drgb), G, ws).cpu().numpy()
    e64, ds64, dc64 = e.astype(np.float64), dsig.astype(np.float64), drgb.astype(np.float64)
    cache = ofield.mlp_fwd(spec, w64, e64, np.abs(e64), ofield.sh_basis(d.astype(np.float64), spec.sh_bands))
    dWs, dWm, de_o, dem = ofield.mlp_bwd(spec, w64, cache, ds64, np.abs(ds64), dc64, np.abs(dc64))
    check_mag("step-edge dL/de", de.transpose(1, 0, 2).reshape(S, 2 * L), de_o, dem, 1e-5)
    _, gws = split_grads(G.cpu().numpy().astype(np.float64), f.layout, spec)
    for j, (a, b, m) in enumerate(zip(gws, dWs, dWm)):
        check_mag(f"step-edge grad W{j}", a, b + 0.5, m + 0.5, 1e-5)


@pytest.mark.parametrize("spec", [W.C1_FIELD, W.C2_FIELD], ids=["tiny", "full"])
@pytest.mark.parametrize("S,k", [(16, 1), (33, 32), (255, 17), (257, 256), (300, 65), (65553, 32769)])
def test_mixed_backward_at_step_edges(nsl, gpu, spec, S, k):
    """nsl_field_bwd_mixed around its tiles of 16 samples, products of 32, steps
    of 256 and rounds of 256 workgroups: the weight gradients of S samples
    against the oracle at 2e-2 of their magnitudes, and against the sum of
    those of the first k and of the others, which differs in the order of FP32
    additions only (1e-5)."""
    import torch
    f = nsl.Field(spec)
    flat, t64, w64 = params_for(spec, f.layout, seed=7, table_range=0.5)
    rng = np.random.default_rng(S)
    xn = rng.uniform(size=(S, 3)).astype(np.float32)
    d = rng.normal(size=(S, 3))
    d = (d / np.linalg.norm(d, axis=1, keepdims=True)).astype(np.float32)
    dsig = rng.normal(size=S).astype(np.float32)
    drgb = rng.normal(size=(S, 3)).astype(np.float32)
    shadow = f.prepare_mixed(_t(torch, gpu, flat))

    def grads(lo, hi):
        G = torch.zeros(f.layout["total"], device=gpu)
        ws = torch.empty(f.workspace_bytes(hi - lo), dtype=torch.uint8, device=gpu)
        f.bwd_mixed(shadow, *(_t(torch, gpu, a[lo:hi]) for a in (xn, d, dsig, drgb)), G, ws)
        return split_grads(G.cpu().numpy().astype(np.float64), f.layout, spec)[1]

    e, em, _ = ofield.encode_fwd(spec, t64, xn)
    cache = ofield.mlp_fwd(spec, w64, e, em, ofield.sh_basis(d.astype(np.float64), spec.sh_bands), band=2e-2)
    ds64, dc64 = dsig.astype(np.float64), drgb.astype(np.float64)
    dWs, dWm, _, _ = ofield.mlp_bwd(spec, w64, cache, ds64, np.abs(ds64), dc64, np.abs(dc64), band_tol=2e-2)
    whole, first, rest = grads(0, S), grads(0, k), grads(k, S)
    for j, (g, a, b, want, m) in enumerate(zip(whole, first, rest, dWs, dWm)):
        check_mag(f"mixed step-edge grad W{j}", g, want, m, 2e-2)
        check_mag(f"mixed step-edge parts W{j}", a + b, g, m, 1e-5)


# four levels of 111 KB in FP32, which the encoding reads from memory, and 56 KB
# in FP16, which it copies to LDS
MID_TABLES = dataclasses.replace(W.C1_FIELD, log2_table=13)


@pytest.mark.parametrize("spec", [W.C1_FIELD, MID_TABLES], ids=["in-lds", "fp16-in-lds"])
@pytest.mark.parametrize("S", [1, 511, 513, 525001])
def test_encode_of_tables_in_lds(nsl, gpu, spec, S):
    """nsl_encode_fwd (1e-5 of the magnitudes) and nsl_encode_fwd_mixed (2e-2)
    around the workgroup's 512 samples and past one round of all workgroups,
    with points outside the box, for tables that fit LDS and one that does not."""
    import torch
    f = nsl.Field(spec)
    flat, t64, _ = params_for(spec, f.layout, seed=10, table_range=0.5)
    xn = np.random.default_rng(S).uniform(-0.02, 1.02, size=(S, 3)).astype(np.float32)
    X, P = _t(torch, gpu, xn), _t(torch, gpu, flat)
    got = nsl.encode_fwd(f, P, X).cpu().numpy()
    half = nsl.encode_fwd_mixed(f, f.prepare_mixed(P), X).view(torch.bfloat16).float().cpu().numpy()
    want, mag, _ = ofield.encode_fwd(spec, t64, np.clip(xn, 0, 1))
    order = lambda a: a.reshape(spec.levels, S, 2).transpose(1, 0, 2).reshape(S, 2 * spec.levels)
    check_mag("encoding", order(got), want, mag, 1e-5)
    check_mag("encoding (mixed)", order(half), want, mag, 2e-2)


@pytest.mark.parametrize("S", [32767, 32768, 32769, 32768 + 63, 40001])
def test_mixed_forward_level_by_level(nsl, gpu, S):
    """nsl_field_fwd_mixed of the 16-level field around the sample count from
    which it gathers level by level: the same bits as calls of fewer samples,
    which gather all levels at once."""
    import torch
    f = nsl.Field(W.C2_FIELD)
    flat, _, _ = params_for(W.C2_FIELD, f.layout, seed=8, table_range=0.5)
    rng = np.random.default_rng(S)
    xn = _t(torch, gpu, rng.uniform(-0.01, 1.01, size=(S, 3)).astype(np.float32))
    d = rng.normal(size=(S, 3))
    d = _t(torch, gpu, (d / np.linalg.norm(d, axis=1, keepdims=True)).astype(np.float32))
    shadow = f.prepare_mixed(_t(torch, gpu, flat))
    sg, rgb = f.fwd_mixed(shadow, xn, d)
    for lo in range(0, S, 16384):
        a, b = f.fwd_mixed(shadow, xn[lo:lo + 16384].contiguous(), d[lo:lo + 16384].contiguous())
        assert torch.equal(sg[lo:lo + 16384], a) and torch.equal(rgb[lo:lo + 16384], b)


@pytest.mark.parametrize("c,p", [(1, 1), (15, 63), (16, 64), (17, 257), (48, 300), (60, 65), (60, 70001)])
def test_covariance_at_tile_edges(nsl, gpu, c, p):
    """nsl_depth_covariance around the 16x16 tiles, the 16-pixel groups, the
    256-pixel chunks and the 256 partial sums, for any c (not only whole
    keyframes), against the oracle in FP64: 1e-9, as the whole-window test."""
    import torch
    rng = np.random.default_rng(100 * c + p)
    E = rng.normal(size=(c, p))
    P = rng.uniform(0.5, 20.0, size=p)
    A = rng.normal(size=(c, c))
    C = (E / P) @ E.T + A @ A.T + 3.0 * np.eye(c)         # H_T = A A^T + 3 I
    d = rng.uniform(0.2, 2.0, size=p)
    sT, sd, dv, st = nsl.depth_covariance(_t(torch, gpu, C), _t(torch, gpu, E.T), _t(torch, gpu, P), _t(torch, gpu, d))
    assert int(st.item()) == 0
    oT, od = ocov.marginals(C, E, P)
    got = sT.cpu().numpy()
    assert np.allclose(got, oT, rtol=1e-9, atol=1e-12 * np.abs(oT).max())
    assert np.array_equal(got, got.T)
    assert np.allclose(sd.cpu().numpy(), od, rtol=1e-9)
    assert np.allclose(dv.cpu().numpy(), ocov.depth_variance(od, d), rtol=1e-6)


def test_covariance_refuses_a_negative_depth_hessian(nsl, gpu):
    """A pixel whose P is negative makes the window indefinite: status 1 and NaN."""
    import torch
    C, E, P, d = W.ba_window(seed=5, n_kf=2, h=3, w=4)
    P[7] = -P[7]
    sT, sd, _, st = nsl.depth_covariance(_t(torch, gpu, C), _t(torch, gpu, E.T), _t(torch, gpu, P), _t(torch, gpu, d))
    assert int(st.item()) == 1 and bool(torch.isnan(sT).all()) and bool(torch.isnan(sd).all())


@pytest.mark.parametrize("n,H,Wd", [(1, 3, 3), (15, 4, 5), (16, 1, 65), (17, 97, 2), (33, 90, 95)])
@pytest.mark.parametrize("spec", [W.C1_FIELD, W.C2_FIELD], ids=["tiny", "full"])
def test_render_at_block_and_round_edges(nsl, gpu, spec, n, H, Wd):
    """nsl_render around its 4x4-pixel blocks, its 16-sample rounds and the
    512-block stretches of an XCD, against the oracle's render at 1e-5 of the
    magnitudes; every pixel written once and nothing else."""
    import torch
    f = nsl.Field(spec)
    flat, t64, w64 = params_for(spec, f.layout, seed=n, table_range=1.0)
    pose = W.look_at_pose((1.4 * np.cos(n), 1.4 * np.sin(n), 0.1)).astype(np.float32)
    intr = np.array([0.9375 * Wd, 0.9375 * Wd, Wd / 2, H / 2], np.float32)
    cfg = nsl.render_config(0.5, 2.0 / n, n, 0.0)
    ws = torch.empty(nsl.render_workspace_bytes(f, H, Wd, cfg), dtype=torch.uint8, device=gpu)
    px = H * Wd
    buf = [torch.full((px + 64, 3), -9.0, device=gpu)] + [torch.full((px + 64,), -9.0, device=gpu) for _ in range(3)]
    nsl.render(f, _t(torch, gpu, flat), _t(torch, gpu, pose.reshape(12)), _t(torch, gpu, intr), H, Wd, cfg, ws, *buf)
    o = ostep.render_image(spec, t64, w64, pose, intr, H, Wd,
                           W.SamplerSpec(mode="uniform", t_near=0.5, t_far=2.5, dt=2.0 / n, n_uniform=n))
    for a, k in zip(buf, ("rgb", "depth_z", "var_z", "opacity")):
        got = a.cpu().numpy()
        assert np.all(got[px:] == -9.0), k
        check_mag(f"render edge {k}", got[:px], o[k], o[f"{k}_mag"], 1e-5)


@pytest.mark.parametrize("stop_T", [0.0, 0.3])
@pytest.mark.parametrize("spec", [W.C1_FIELD, W.C2_FIELD], ids=["tiny", "full"])
def test_render_tiles_equal_the_whole_image(nsl, gpu, spec, stop_T):
    """Ragged tiles of 1 to 64 pixels (groups of 16 that are full, partial and
    empty, groups that stop in different rounds) give the pixels of nsl_render,
    bit for bit."""
    import torch
    f = nsl.Field(spec)
    H, Wd, n = 23, 31, 40
    flat, _, _ = params_for(spec, f.layout, seed=2, table_range=2.0)
    P = _t(torch, gpu, flat)
    pose = W.look_at_pose((1.5, 0.3, 0.2)).astype(np.float32)
    intr = np.array([0.9375 * Wd, 0.9375 * Wd, Wd / 2, H / 2], np.float32)
    cfg = nsl.render_config(0.5, 2.0 / n, n, stop_T)
    new = lambda: [torch.full((H * Wd, 3), -9.0, device=gpu)] + [torch.full((H * Wd,), -9.0, device=gpu) for _ in range(3)]
    whole, tiled = new(), new()
    ws = torch.empty(nsl.render_workspace_bytes(f, H, Wd, cfg), dtype=torch.uint8, device=gpu)
    nsl.render(f, P, _t(torch, gpu, pose.reshape(12)), _t(torch, gpu, intr), H, Wd, cfg, ws, *whole)
    prep = nsl.prepare(f, P)
    rng = np.random.default_rng(3)
    tiles, p = [], 0
    while p < H * Wd:
        k = int(rng.choice([1, 15, 16, 17, 31, 33, 48, 49, 64]))
        tiles.append(nsl.RenderTile(0, p, k))
        p += k
    rq = nsl.records_to_device([nsl.render_request(P, prep, pose.reshape(12), intr, H, Wd, *tiled)],
                               nsl.RenderRequest, gpu)
    nsl.render_batch(f, rq, 1, nsl.records_to_device(tiles, nsl.RenderTile, gpu), len(tiles), cfg)
    for a, b in zip(whole, tiled):
        assert torch.equal(a, b)


@pytest.mark.parametrize("bad", [np.inf, -np.inf, np.nan, 3.4e38])
@pytest.mark.parametrize("where", ["table", "first", "hidden"])
def test_render_of_values_that_are_not_finite(nsl, gpu, bad, where):
    """One value of the 16-level field that is not finite (or above the largest
    BF16), in the table or in a weight: the rendered pixels have the same
    finite, infinite and NaN pattern, and the same finite values within 1e-4, as
    compositing the FP32 field's own densities and colours."""
    import torch
    spec = W.C2_FIELD
    f = nsl.Field(spec)
    lay = f.layout
    H, Wd, n = 12, 16, 24
    flat, _, _ = params_for(spec, lay, seed=9, table_range=0.5)
    at = {"table": 2 * (lay["level_offset"][1] + 23 * 23 * 11 + 23 * 11 + 11), "first": lay["w_offsets"][0] + 5,
          "hidden": lay["w_offsets"][3] + 77}[where]
    if where == "table":
        flat[at - 2:at + 4] = bad                       # vertices in the middle of the scene
    else:
        flat[at] = bad
    P = _t(torch, gpu, flat)
    pose = W.look_at_pose((1.5, 0.2, 0.1)).astype(np.float32)
    intr = np.array([0.9375 * Wd, 0.9375 * Wd, Wd / 2, H / 2], np.float32)
    dt = np.float32(2.0 / n)
    cfg = nsl.render_config(0.5, float(dt), n, 0.0)
    ws = torch.empty(nsl.render_workspace_bytes(f, H, Wd, cfg), dtype=torch.uint8, device=gpu)
    op = torch.empty(H * Wd, device=gpu)
    rgb, _, _, _ = nsl.render(f, P, _t(torch, gpu, pose.reshape(12)), _t(torch, gpu, intr), H, Wd, cfg, ws, opacity=op)
    from oracle import rays as orays
    o32, d32, _ = orays.rays_fp32(pose[None], intr[None], np.arange(H * Wd, dtype=np.uint32), H, Wd)
    t = np.float32(0.5) + (np.arange(n, dtype=np.float32) + np.float32(0.5)) * dt
    x = o32[:, None] + t[None, :, None] * d32[:, None]
    xn = np.clip((x + np.float32(1)) * np.float32(0.5), 0, 1).astype(np.float32).reshape(-1, 3)
    S = len(xn)
    fw = torch.empty(f.workspace_bytes(S), dtype=torch.uint8, device=gpu)
    sg, col = f.fwd(P, _t(torch, gpu, xn), _t(torch, gpu, np.repeat(d32, n, 0).astype(np.float32)), fw)
    with np.errstate(all="ignore"):
        tau = sg.cpu().numpy().reshape(-1, n).astype(np.float64) * float(dt)
        before = np.concatenate([np.zeros((len(tau), 1)), np.cumsum(tau, 1)[:, :-1]], 1)
        w = np.exp(-before) * -np.expm1(-tau)
        want = (w[..., None] * col.cpu().numpy().reshape(-1, n, 3)).sum(1)
        opw = w.sum(1)
    for got, ref in ((rgb.cpu().numpy(), want), (op.cpu().numpy(), opw)):
        assert np.array_equal(np.isnan(got), np.isnan(ref))
        ok = np.isfinite(ref)
        assert ok.any() or where != "table"
        assert np.allclose(got[ok], ref[ok], rtol=1e-4, atol=1e-6)


def test_render_of_vanishing_densities(nsl, gpu):
    """Every density about 1e-38, so that a sample's weight is below the
    smallest number with a reciprocal: depth and depth variance, whose running
    mean divides by the weights' sum, stay finite and tiny."""
    import torch
    spec = W.C1_FIELD
    f = nsl.Field(spec)
    H, Wd, n = 24, 32, 16
    flat, _, _ = params_for(spec, f.layout, seed=3, table_range=0.5)
    flat[:f.layout["table_floats"]] = 0.3                 # one encoding, so one density, everywhere
    w1 = flat[f.layout["w_offsets"][1]:][:spec.density_hidden * spec.geo_dim].reshape(-1, spec.geo_dim)
    w1[:, 0] = -np.abs(w1[:, 0])
    xn = np.random.default_rng(1).uniform(size=(256, 3)).astype(np.float32)
    ws = torch.empty(f.workspace_bytes(len(xn)), dtype=torch.uint8, device=gpu)
    X, D = _t(torch, gpu, xn), _t(torch, gpu, np.tile(np.float32([0, 0, 1]), (len(xn), 1)))
    o = np.log(f.fwd(_t(torch, gpu, flat), X, D, ws)[0].cpu().numpy().astype(np.float64))
    w1[:, 0] *= np.float32(-87.0 / np.median(o))
    P = _t(torch, gpu, flat)
    dt = 2.0 / n
    sg = f.fwd(P, X, D, ws)[0].cpu().numpy().astype(np.float64)
    assert np.all(sg > 0) and np.all(sg * dt < 2.0 ** -128)
    cfg = nsl.render_config(0.5, dt, n, 0.0)
    rw = torch.empty(nsl.render_workspace_bytes(f, H, Wd, cfg), dtype=torch.uint8, device=gpu)
    pose = W.look_at_pose((1.5, 0.2, 0.1)).astype(np.float32).reshape(12)
    intr = np.array([0.9375 * Wd, 0.9375 * Wd, Wd / 2, H / 2], np.float32)
    rgb, dz, vz, _ = nsl.render(f, P, _t(torch, gpu, pose), _t(torch, gpu, intr), H, Wd, cfg, rw)
    for a in (rgb, dz, vz):
        a = a.cpu().numpy()
        assert np.all(np.isfinite(a)) and np.all(a >= 0) and np.all(a < 1e-30)


@pytest.mark.parametrize("n,shift", [(16385, 0), (24576, 0), (24577, 1), (40003, 3)])
def test_march_scan_at_segment_edges(nsl, gpu, n, shift):
    """nsl_march of more candidates than the sample emission scans itself,
    around the scan's segments of 8192, with the caller's offsets at any
    4-byte address: counts, offsets and statistics against their definition."""
    import torch
    from parity import upload_keyframes
    kf = W.c1_keyframes()
    f = nsl.Field(W.C1_FIELD)
    m = upload_keyframes(nsl, torch, kf, gpu)
    ids = np.random.default_rng(n).integers(0, 1100, size=n).astype(np.uint32)     # 1024 pixels are stored
    cfg = nsl.step_config(W.C1_SAMPLER)
    ws = torch.empty(nsl.step_workspace_bytes(f, cfg, n), dtype=torch.uint8, device=gpu)
    counts = torch.zeros(n, dtype=torch.int32, device=gpu)
    offs = torch.zeros(n + 1 + shift, dtype=torch.int32, device=gpu)[shift:]
    t = torch.zeros(cfg.max_samples, dtype=torch.float32, device=gpu)
    ray = torch.zeros(cfg.max_samples, dtype=torch.int32, device=gpu)
    stats = torch.zeros(4, dtype=torch.int32, device=gpu)
    nsl.march(m, f, cfg, _t(torch, gpu, ids.view(np.int32)), ws, counts, offs, t, ray, stats)
    want = np.where(ids < 1024, 32, 0)
    ends = np.cumsum(want)
    kept = ends <= cfg.max_samples
    assert np.array_equal(counts.cpu().numpy(), want)
    assert np.array_equal(offs.cpu().numpy(), np.concatenate([[0], ends]))
    got = stats.cpu().numpy()
    assert got[:3].tolist() == [int(np.sum(kept & (want > 0))), int(ends[kept].max()), int(kept.sum())]
    assert np.array_equal(ray.cpu().numpy()[:got[1]], np.repeat(np.arange(n), want)[:got[1]])


@pytest.mark.parametrize("n_uniform", [1, 16, 17, 31, 32, 33])
def test_step_of_short_rays(nsl, gpu, n_uniform):
    """An FP32 step of an odd number of candidates, one of them no stored pixel
    and the last ones cut off, around the 32 samples a ray up to which two rays
    share a wave in the compositing: every output and gradient at 1e-5."""
    import torch
    from test_gpu_parity import _compare_step, _step_gpu
    sampler = dataclasses.replace(W.C1_SAMPLER, n_uniform=n_uniform, dt=2.0 / n_uniform,
                                  max_samples=n_uniform * 997 + n_uniform // 2)
    spec, kf = W.C1_FIELD, W.c1_keyframes()
    ids = np.concatenate([W.c1_pixels()[:500], np.array([5000], np.uint32), W.c1_pixels()[500:1000]])
    f = nsl.Field(spec)
    flat, t64, w64 = params_for(spec, f.layout, seed=11, table_range=0.2)
    stored = ids < 1024
    o = ostep.train_step(spec, sampler, kf, t64, w64, ids[stored])
    g = _step_gpu(nsl, torch, gpu, spec, sampler, kf, ids, flat)
    assert np.all(g["rays"][~stored] == 0)
    g["rays"] = g["rays"][stored]
    _compare_step(spec, g, o, f.layout, tol=1e-5)


@pytest.mark.parametrize("R", [1, 7, 1001])
def test_composite_adjoint_of_rows(nsl, gpu, R):
    """nsl_composite_bwd_rows gives the bits of nsl_composite_bwd with the
    columns of its seeds; a gradient of another shape is refused, one that is
    expanded or transposed differentiates the same."""
    import torch
    from paper_2210_13641_amd import autograd as ag
    rng = np.random.default_rng(R)
    n = rng.integers(0, 90, R)
    off = _t(torch, gpu, np.concatenate([[0], np.cumsum(n)]).astype(np.int32))
    S = max(1, int(n.sum()))
    sg = _t(torch, gpu, np.exp(rng.normal(size=S)).astype(np.float32))
    rgb = _t(torch, gpu, rng.uniform(size=(S, 3)).astype(np.float32))
    t = _t(torch, gpu, np.sort(rng.uniform(0.5, 2.5, S)).astype(np.float32))
    g = _t(torch, gpu, rng.normal(size=(R, 6)).astype(np.float32))
    cols = (g[:, :3].contiguous(), *(g[:, k].contiguous() for k in (3, 4, 5)))
    want = nsl.composite_bwd(sg, rgb, t, off, 0.03, *cols)
    for seeds in (g, g.t().contiguous().t()):
        a, b = sg.clone().requires_grad_(True), rgb.clone().requires_grad_(True)
        ag.CompositeFunction.apply(a, b, t, off, 0.03).backward(seeds)
        assert torch.equal(a.grad, want[0]) and torch.equal(b.grad, want[1])
    a = sg.clone().requires_grad_(True)
    ag.CompositeFunction.apply(a, rgb, t, off, 0.03).sum().backward()       # an expanded gradient
    one = nsl.composite_bwd_rows(sg, rgb, t, off, 0.03, torch.ones(R, 6, device=gpu))
    assert torch.equal(a.grad, one[0])
    with pytest.raises(ValueError):
        nsl.composite_bwd_rows(sg, rgb, t, off, 0.03, g[:, :3].contiguous())


@pytest.mark.parametrize("spec", [W.C1_FIELD, W.C2_FIELD], ids=["tiny", "full"])
@pytest.mark.parametrize("n", [32, 64])
def test_render_depth_variance_error(nsl, gpu, spec, n):
    """V* of rays of constant density 1 (a field of zeros) against FP64: the
    mean relative error over 400 rays of different t_near and dt stays below
    8e-8.  Weights and t rounded to FP32 with V* summed exactly give 3.6e-8
    (32 samples) and 4.5e-8 (64), with the sum about the final d* in FP32
    7.0e-8 and 7.2e-8."""
    import torch
    f = nsl.Field(spec)
    P = torch.zeros(f.layout["total"], device=gpu)
    pose = _t(torch, gpu, W.look_at_pose((1.5, 0.0, 0.0)).astype(np.float32).reshape(12))
    intr = _t(torch, gpu, np.array([1.0, 1.0, 0.5, 0.5], np.float32))    # the pixel looks straight ahead: s = 1
    rng = np.random.default_rng(n)
    j = np.arange(n, dtype=np.float32) + np.float32(0.5)
    got, want = [], []
    ws = None
    for _ in range(400):
        near, dt = np.float32(rng.uniform(0.05, 2.0)), np.float32(np.exp(rng.uniform(np.log(0.01), np.log(0.3))))
        cfg = nsl.render_config(float(near), float(dt), n, 0.0)
        if ws is None:
            ws = torch.empty(nsl.render_workspace_bytes(f, 1, 1, cfg), dtype=torch.uint8, device=gpu)
        got.append(nsl.render(f, P, pose, intr, 1, 1, cfg, ws)[2])
        t = (near + j * dt).astype(np.float64)
        w = np.exp(-np.float64(dt) * np.arange(n)) * -np.expm1(-np.float64(dt))
        want.append((w * (t - (w * t).sum()) ** 2).sum())
    err = np.abs(torch.cat(got).cpu().numpy().astype(np.float64) / np.array(want) - 1.0)
    assert err.mean() < 8e-8, err.mean()


@pytest.mark.parametrize("stop_T", [0.0, 0.3])
@pytest.mark.parametrize("spec,n", [(W.C1_FIELD, 1), (W.C1_FIELD, 17), (W.C1_FIELD, 300), (W.C2_FIELD, 40),
                                    (W.C2_FIELD, 300)], ids=["tiny-1", "tiny-17", "tiny-300", "full-40", "full-300"])
def test_render_of_few_pixels_equals_the_whole_image(nsl, gpu, spec, n, stop_T):
    """Groups of 1 to 16 pixels, whose tiles hold 16 to 1 samples of a ray,
    give the pixels of nsl_render bit for bit: one pass over a ray and several,
    images whose edges are groups of one to four columns or rows, of one pixel,
    one row and one column."""
    import torch
    f = nsl.Field(spec)
    flat, _, _ = params_for(spec, f.layout, seed=n, table_range=2.0)
    P = _t(torch, gpu, flat)
    prep = nsl.prepare(f, P)
    pose = W.look_at_pose((1.5, 0.3, 0.2)).astype(np.float32).reshape(12)
    cfg = nsl.render_config(0.5, 2.0 / n, n, stop_T)
    rng = np.random.default_rng(n)
    for H, Wd in ((1, 1), (1, 37), (33, 1), (2, 19), (7, 13)):
        intr = np.array([12.0, 12.0, Wd / 2, H / 2], np.float32)
        new = lambda: [torch.full((H * Wd, 3), -9.0, device=gpu)] + [torch.full((H * Wd,), -9.0, device=gpu) for _ in range(3)]
        whole, tiled = new(), new()
        ws = torch.empty(nsl.render_workspace_bytes(f, H, Wd, cfg), dtype=torch.uint8, device=gpu)
        nsl.render(f, P, _t(torch, gpu, pose), _t(torch, gpu, intr), H, Wd, cfg, ws, *whole)
        assert all(bool((a != -9.0).all()) for a in whole)
        tiles, p = [], 0
        while p < H * Wd:
            k = int(rng.integers(1, 20))
            tiles.append(nsl.RenderTile(0, p, k))
            p += k
        rq = nsl.records_to_device([nsl.render_request(P, prep, pose, intr, H, Wd, *tiled)], nsl.RenderRequest, gpu)
        nsl.render_batch(f, rq, 1, nsl.records_to_device(tiles, nsl.RenderTile, gpu), len(tiles), cfg)
        for a, b in zip(whole, tiled):
            assert torch.equal(a, b), (H, Wd)


def _shortest_ms(torch, call, n=8):
    """The shortest of seven timings of n calls, per call."""
    a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    best = np.inf
    for _ in range(8):                      # (the first warms up: it is longer)
        a.record()
        for _ in range(n):
            call()
        b.record()
        b.synchronize()
        best = min(best, a.elapsed_time(b) / n)
    return best


def test_render_of_one_row_costs_its_pixels(nsl, gpu):
    """16384 pixels in one row or one column take at most twice the time of a
    128x128 image (about as long; three times as long when every 4x4 block evaluated
    the pixels it does not have)."""
    import torch
    f = nsl.Field(W.C1_FIELD)
    P = _t(torch, gpu, params_for(W.C1_FIELD, f.layout, seed=1, table_range=0.2)[0])
    pose = _t(torch, gpu, W.look_at_pose((1.5, 0.2, 0.1)).astype(np.float32).reshape(12))
    cfg = nsl.render_config(0.5, 2.0 / 64, 64, 0.0)

    def ms(H, Wd):
        s = 0.9375 * max(H, Wd)
        intr = _t(torch, gpu, np.array([s, s, Wd / 2, H / 2], np.float32))
        ws = torch.empty(nsl.render_workspace_bytes(f, H, Wd, cfg), dtype=torch.uint8, device=gpu)
        return _shortest_ms(torch, lambda: nsl.render(f, P, pose, intr, H, Wd, cfg, ws))

    square = ms(128, 128)
    assert ms(1, 16384) < 2.0 * square and ms(16384, 1) < 2.0 * square


@pytest.mark.parametrize("spec", [W.C1_FIELD, W.C2_FIELD], ids=["tiny", "full"])
def test_render_of_ragged_tiles_costs_their_pixels(nsl, gpu, spec):
    """A 160x120 image by tiles of 1 or 16 pixels takes at most twice the time it
    takes by tiles of 64 (measured 0.9 to 1.7 times; with each tile's first 16 pixels
    on one fourth of the CUs 2.3 to 5.3)."""
    import torch
    f = nsl.Field(spec)
    H, Wd, n = 120, 160, 64
    P = _t(torch, gpu, params_for(spec, f.layout, seed=1, table_range=0.2)[0])
    prep = nsl.prepare(f, P)
    out = [torch.empty(H * Wd, 3, device=gpu)] + [torch.empty(H * Wd, device=gpu) for _ in range(3)]
    pose = W.look_at_pose((1.5, 0.2, 0.1)).astype(np.float32).reshape(12)
    rq = nsl.records_to_device([nsl.render_request(P, prep, pose, [150.0, 150.0, 80.0, 60.0], H, Wd, *out)],
                               nsl.RenderRequest, gpu)
    cfg = nsl.render_config(0.5, 2.0 / n, n, 0.0)

    def ms(k):
        tiles = [nsl.RenderTile(0, p, k) for p in range(0, H * Wd, k)]
        td = nsl.records_to_device(tiles, nsl.RenderTile, gpu)
        return _shortest_ms(torch, lambda: nsl.render_batch(f, rq, 1, td, len(tiles), cfg))

    whole = ms(64)
    assert ms(16) < 2.0 * whole and ms(1) < 2.0 * whole


def test_render_of_a_small_image_spreads_over_the_chip(nsl, gpu):
    """4x4 pixels of the 64-wide network take at most three times as long as one
    (1.3 times; 6.7 times as one group of 16, whose 64 tiles four waves share)."""
    import torch
    f = nsl.Field(W.C2_FIELD)
    P = _t(torch, gpu, params_for(W.C2_FIELD, f.layout, seed=1, table_range=0.2)[0])
    pose = _t(torch, gpu, W.look_at_pose((1.5, 0.2, 0.1)).astype(np.float32).reshape(12))
    cfg = nsl.render_config(0.5, 2.0 / 64, 64, 0.0)

    def ms(side):
        intr = _t(torch, gpu, np.array([side, side, side / 2, side / 2], np.float32))
        ws = torch.empty(nsl.render_workspace_bytes(f, side, side, cfg), dtype=torch.uint8, device=gpu)
        return _shortest_ms(torch, lambda: nsl.render(f, P, pose, intr, side, side, cfg, ws))

    assert ms(4) < 3.0 * ms(1)


def test_render_beside_values_that_are_not_finite(nsl, gpu):
    """Infinite entries of the 16-level field's table: the pixels whose rays stay
    clear of their cells keep the bits of the render without them, those in a
    4x4 block with a touched one included."""
    import torch
    from oracle import rays as orays
    spec = W.C2_FIELD
    f = nsl.Field(spec)
    H, Wd, n = 160, 160, 12                              # 1600 blocks of 4x4
    flat, _, _ = params_for(spec, f.layout, seed=9, table_range=2.0)
    bad = flat.copy()
    at = 2 * (f.layout["level_offset"][1] + 23 * 23 * 11 + 23 * 11 + 11)     # level 1: 22 cells an axis
    bad[at - 2:at + 4] = np.inf                          # vertices x = 10, 11, 12 of y = z = 11
    pose = W.look_at_pose((1.5, 0.2, 0.1)).astype(np.float32)
    intr = np.array([150.0, 150.0, Wd / 2, H / 2], np.float32)
    dt = np.float32(2.0 / n)
    cfg = nsl.render_config(0.5, float(dt), n, 0.0)
    ws = torch.empty(nsl.render_workspace_bytes(f, H, Wd, cfg), dtype=torch.uint8, device=gpu)
    out = []
    for p in (flat, bad):
        op = torch.empty(H * Wd, device=gpu)
        r = nsl.render(f, _t(torch, gpu, p), _t(torch, gpu, pose.reshape(12)), _t(torch, gpu, intr), H, Wd, cfg, ws,
                       opacity=op)
        out.append(np.concatenate([a.cpu().numpy().reshape(H * Wd, -1) for a in r], 1))
    o32, d32, _ = orays.rays_fp32(pose[None], intr[None], np.arange(H * Wd, dtype=np.uint32), H, Wd)
    t = np.float32(0.5) + (np.arange(n, dtype=np.float32) + np.float32(0.5)) * dt
    cell = np.clip((o32[:, None] + t[None, :, None] * d32[:, None] + 1.0) * 0.5, 0, 1) * 22
    lo, hi = np.array([9, 10, 10]), np.array([13, 12, 12])
    near = ((cell > lo - 1e-3) & (cell < hi + 1e-3)).all(-1).any(-1)
    inside = ((cell > lo + 1e-3) & (cell < hi - 1e-3)).all(-1).any(-1)
    assert not np.isfinite(out[1][inside]).all(-1).any()
    block = near.reshape(H // 4, 4, Wd // 4, 4).any((1, 3)).repeat(4, 0).repeat(4, 1).reshape(-1)
    assert np.sum(block & ~near) > 100                   # clear pixels beside touched ones
    assert np.array_equal(out[0][~near].view(np.int32), out[1][~near].view(np.int32))


@pytest.mark.parametrize("spec", [W.C1_FIELD, W.C2_FIELD], ids=["tiny", "full"])
@pytest.mark.parametrize("S", [1, 4097, 19999, 20000, 40001])
def test_field_forward_leaves_the_records_alone(nsl, gpu, spec, S):
    """nsl_field_fwd and Field.fwd write the weight operands of their workspace
    and nothing behind them, where a backward on another stream may hold its
    encoding or records; and both give the bits of calls of fewer samples, around
    the count from which Field.fwd encodes apart."""
    import torch
    f = nsl.Field(spec)
    flat, _, _ = params_for(spec, f.layout, seed=12, table_range=0.5)
    P = _t(torch, gpu, flat)
    rng = np.random.default_rng(S)
    X = _t(torch, gpu, rng.uniform(-0.01, 1.01, size=(S, 3)).astype(np.float32))
    d = rng.normal(size=(S, 3))
    D = _t(torch, gpu, (d / np.linalg.norm(d, axis=1, keepdims=True)).astype(np.float32))
    ws = torch.full((f.workspace_bytes(S),), 0xA5, dtype=torch.uint8, device=gpu)
    sg, rgb = f.fwd(P, X, D, ws)
    sg2, rgb2 = torch.empty_like(sg), torch.empty_like(rgb)
    assert nsl._lib.nsl_field_fwd(f.handle, P.data_ptr(), X.data_ptr(), D.data_ptr(), S, sg2.data_ptr(),
                                  rgb2.data_ptr(), ws.data_ptr(), ws.numel(), nsl._stream()) == 0
    assert bool((ws[nsl.prepared_bytes(f):] == 0xA5).all())
    assert torch.equal(sg, sg2) and torch.equal(rgb, rgb2)
    for lo in range(0, S, 16384):
        a, b = f.fwd(P, X[lo:lo + 16384].contiguous(), D[lo:lo + 16384].contiguous(), ws)
        assert torch.equal(sg[lo:lo + 16384], a) and torch.equal(rgb[lo:lo + 16384], b)


@pytest.mark.parametrize("n,n_uniform,shift", [(16386, 32, 1), (40003, 32, 2), (24576, 32, 3), (1 << 20, 4096, 0),
                                               ((1 << 20) + 70001, 4096, 1)])
def test_march_scan_of_any_counts(nsl, gpu, n, n_uniform, shift):
    """nsl_march with the caller's counts at any 4-byte address, and with 2^32
    samples and more before the cut: a wrapped offset would start over below
    max_samples.  Every candidate's offset is the exact prefix as far as 32 bits
    less 2^26 go, and the kept ones are a prefix."""
    import torch
    from parity import upload_keyframes
    f = nsl.Field(W.C1_FIELD)
    m = upload_keyframes(nsl, torch, W.c1_keyframes(), gpu)
    ids = np.random.default_rng(n).integers(0, 1100 if n < 1 << 20 else 1024, size=n).astype(np.uint32)
    cfg = nsl.step_config(dataclasses.replace(W.C1_SAMPLER, n_uniform=n_uniform, max_samples=70000))
    ws = torch.empty(nsl.step_workspace_bytes(f, cfg, n), dtype=torch.uint8, device=gpu)
    counts = torch.zeros(n + shift, dtype=torch.int32, device=gpu)[shift:]
    offs = torch.zeros(n + 1, dtype=torch.int32, device=gpu)
    t = torch.zeros(cfg.max_samples, dtype=torch.float32, device=gpu)
    ray = torch.full((cfg.max_samples,), -1, dtype=torch.int32, device=gpu)
    stats = torch.zeros(4, dtype=torch.int32, device=gpu)
    nsl.march(m, f, cfg, _t(torch, gpu, ids.view(np.int32)), ws, counts, offs, t, ray, stats)
    want = np.where(ids < 1024, n_uniform, 0).astype(np.int64)
    ends = np.cumsum(want)
    kept = ends <= cfg.max_samples
    cap = 2 ** 32 - 1 - 2 ** 26
    assert np.array_equal(counts.cpu().numpy(), want)
    assert np.array_equal(offs.cpu().numpy().view(np.uint32), np.minimum(np.concatenate([[0], ends]), cap))
    got = stats.cpu().numpy()
    assert got[:3].tolist() == [int(np.sum(kept & (want > 0))), int(ends[kept].max()), int(kept.sum())]
    own = ray.cpu().numpy()
    assert np.array_equal(own[:got[1]], np.repeat(np.arange(n), want)[:got[1]] if n < 1 << 20 else
                          np.arange(got[1]) // n_uniform)
    assert np.all(own[got[1]:] == -1)


# four levels whose table does not fit LDS in FP16 either, the last one of several bins
WIDE_TABLES = dataclasses.replace(W.C1_FIELD, log2_table=15)


def _same_step(a, b, nt):
    """Two steps with the same encoding: the same bits but for the order of the
    table-gradient sums."""
    assert np.array_equal(a["stats"], b["stats"]) and np.array_equal(a["loss"], b["loss"])
    assert np.array_equal(a["rays"], b["rays"])
    assert np.array_equal(a["grads"][nt:], b["grads"][nt:])
    ga, gb = a["grads"][:nt].astype(np.float64), b["grads"][:nt].astype(np.float64)
    assert np.count_nonzero(ga) > 0.1 * nt
    assert np.allclose(ga, gb, rtol=1e-5, atol=1e-6 * np.abs(ga).max())


@pytest.mark.parametrize("mixed", [False, True], ids=["fp32", "mixed"])
@pytest.mark.parametrize("spec", [W.C1_FIELD, MID_TABLES, WIDE_TABLES], ids=["in-lds", "fp16-in-lds", "in-memory"])
def test_step_of_four_levels_with_and_without_kept_encoding(nsl, gpu, spec, mixed):
    """The 4-level field gathers its table in the network's kernels, or with the
    encoding kept in a launch before them (from LDS, or level by level, which also
    counts the table-gradient records): the same step either way."""
    import torch
    from test_gpu_parity import _step_gpu
    f = nsl.Field(spec)
    flat, _, _ = params_for(spec, f.layout, seed=13, table_range=0.3)
    kf, ids = W.c1_keyframes(), W.c1_pixels()
    a, b = [_step_gpu(nsl, torch, gpu, spec, W.C1_SAMPLER, kf, ids, flat, keep_encoding=k, mixed=mixed)
            for k in (False, True)]
    _same_step(a, b, f.layout["table_floats"])


SMALL_SCENE = dataclasses.replace(SMALL_TABLES, aabb_min=(-2.0,) * 3, aabb_max=(2.0,) * 3)


@pytest.mark.parametrize("keep", [False, True], ids=["shared", "kept"])
def test_step_of_sixteen_single_bin_levels(nsl, gpu, keep):
    """A step of 16 levels that each fit one bin, whose encoding (not kept) and
    sums over the parts of the samples lie in one region in turn: loss, outputs,
    table and weight gradients against the oracle at 1e-5; in mixed precision the
    same step with the encoding in that region and in its own."""
    import torch
    from test_gpu_parity import _compare_step, _step_gpu
    spec, kf, ids = SMALL_SCENE, W.c1_keyframes(), W.c1_pixels()
    f = nsl.Field(spec)
    flat, t64, w64 = params_for(spec, f.layout, seed=14, table_range=0.2)
    g = _step_gpu(nsl, torch, gpu, spec, W.C1_SAMPLER, kf, ids, flat, keep_encoding=keep)
    _compare_step(spec, g, ostep.train_step(spec, W.C1_SAMPLER, kf, t64, w64, ids), f.layout, tol=1e-5)
    if keep:
        a, b = [_step_gpu(nsl, torch, gpu, spec, W.C1_SAMPLER, kf, ids, flat, keep_encoding=k, mixed=True)
                for k in (False, True)]
        _same_step(a, b, f.layout["table_floats"])


@pytest.mark.parametrize("S", [16, 700, 20001])
def test_field_backward_of_sixteen_single_bin_levels(nsl, gpu, S):
    """nsl_field_bwd (1e-5) and nsl_field_bwd_mixed (2e-2) of the same field against
    the oracle: the counting sort (too few samples for a part), one part and several."""
    import torch
    spec = SMALL_SCENE
    f = nsl.Field(spec)
    flat, t64, w64 = params_for(spec, f.layout, seed=15, table_range=0.5)
    rng = np.random.default_rng(S)
    xn = rng.uniform(size=(S, 3)).astype(np.float32)
    d = rng.normal(size=(S, 3))
    d = (d / np.linalg.norm(d, axis=1, keepdims=True)).astype(np.float32)
    dsig, drgb = rng.normal(size=S).astype(np.float32), rng.normal(size=(S, 3)).astype(np.float32)
    P = _t(torch, gpu, flat)
    args = [_t(torch, gpu, a) for a in (xn, d, dsig, drgb)]
    ws = torch.empty(f.workspace_bytes(S), dtype=torch.uint8, device=gpu)
    e, em, corners = ofield.encode_fwd(spec, t64, xn)
    sh = ofield.sh_basis(d.astype(np.float64), spec.sh_bands)
    for mixed, tol in ((False, 1e-5), (True, 2e-2)):
        G = torch.zeros(f.layout["total"], device=gpu)
        f.bwd_mixed(f.prepare_mixed(P), *args, G, ws) if mixed else f.bwd(P, *args, G, ws)
        cache = ofield.mlp_fwd(spec, w64, e, em, sh, band=tol)
        ds64, dc64 = dsig.astype(np.float64), drgb.astype(np.float64)
        dWs, dWm, de, dem = ofield.mlp_bwd(spec, w64, cache, ds64, np.abs(ds64), dc64, np.abs(dc64), band_tol=tol)
        gt, gtm = ofield.encode_bwd(spec, corners, de, dem, f.layout["table_floats"])
        tab, gws = split_grads(G.cpu().numpy(), f.layout, spec)
        check_mag(f"small 16-level table gradient {mixed}", tab, gt, gtm, tol)
        for j, (a, b, m) in enumerate(zip(gws, dWs, dWm)):
            check_mag(f"small 16-level grad W{j} {mixed}", a, b, m, tol)


@pytest.mark.parametrize("log2_table", [19, 21])
@pytest.mark.parametrize("S", [255, 20001])
def test_field_backward_counts_as_the_layers_do(nsl, gpu, S, log2_table):
    """nsl_field_bwd of the 16-level field, whose encoding counts the
    table-gradient records (2^19 entries a level; 2^21, which fill the 256 bins it
    counts at most), against nsl_encode_fwd, nsl_mlp_bwd and nsl_encode_bwd, which counts them in a
    pass of its own: the weight gradients bit for bit, the table's up to the order
    of its sums."""
    import torch
    spec = dataclasses.replace(W.C2_FIELD, log2_table=log2_table)
    f = nsl.Field(spec)
    nt = f.layout["table_floats"]
    rng = np.random.default_rng(S)
    P = _t(torch, gpu, params_for(spec, f.layout, seed=16, table_range=0.5)[0])
    o, step = rng.uniform(0.2, 0.8, size=(S // 32 + 1, 1, 3)), rng.normal(size=(S // 32 + 1, 1, 3)) * 0.003
    xn = (o + step * np.arange(32)[:, None]).clip(0, 1).reshape(-1, 3)[:S]       # samples along rays share cells
    d = rng.normal(size=(S, 3))
    X, D = _t(torch, gpu, xn.astype(np.float32)), _t(torch, gpu, (d / np.linalg.norm(d, axis=1, keepdims=True)).astype(np.float32))
    ds, dc = _t(torch, gpu, rng.normal(size=S).astype(np.float32)), _t(torch, gpu, rng.normal(size=(S, 3)).astype(np.float32))
    ws = torch.empty(f.workspace_bytes(S), dtype=torch.uint8, device=gpu)
    a, b = torch.zeros_like(P), torch.zeros_like(P)
    f.bwd(P, X, D, ds, dc, a, ws)
    nsl.encode_bwd(f, X, nsl.mlp_bwd(f, P, nsl.encode_fwd(f, P, X), D, ds, dc, b, ws), b)
    assert torch.equal(a[nt:], b[nt:])
    ga, gb = a[:nt].cpu().numpy().astype(np.float64), b[:nt].cpu().numpy().astype(np.float64)
    assert np.array_equal(ga != 0, gb != 0) and np.count_nonzero(ga) > 0
    assert np.allclose(ga, gb, rtol=1e-5, atol=1e-6 * np.abs(ga).max())


@pytest.mark.parametrize("bad", [np.inf, -np.inf, np.nan])
@pytest.mark.parametrize("n_uniform", [32, 33])
def test_step_keeps_bad_densities_to_their_rays(nsl, gpu, bad, n_uniform):
    """A vertex of the tiny field's table that is not finite, in the compositing
    of two rays a wave (32 samples) and of one (33): the outputs of the rays clear
    of its cells keep their bits, beside touched rays in the same wave."""
    import torch
    from oracle import rays as orays
    from test_gpu_parity import _step_gpu
    spec, kf, ids = W.C1_FIELD, W.c1_keyframes(), W.c1_pixels()
    sampler = dataclasses.replace(W.C1_SAMPLER, n_uniform=n_uniform, dt=2.0 / n_uniform)
    f = nsl.Field(spec)
    flat, _, _ = params_for(spec, f.layout, seed=17, table_range=0.3)
    hurt = flat.copy()
    at = 2 * (f.layout["level_offset"][1] + (4 * 9 + 4) * 9 + 4)          # level 1: 8 cells an axis
    hurt[at:at + 2] = bad
    a, b = [_step_gpu(nsl, torch, gpu, spec, sampler, kf, ids, p)["rays"] for p in (flat, hurt)]
    o32, d32, _ = orays.rays_fp32(kf.pose, kf.intr, ids, 32, 32)
    t = orays.uniform_t(sampler)
    cell = np.clip((o32[:, None] + t[None, :, None] * d32[:, None] + 2.0) / 4.0, 0, 1) * 8
    near = ((cell > 3 - 1e-3) & (cell < 5 + 1e-3)).all(-1).any(-1)
    inside = ((cell > 3 + 1e-3) & (cell < 5 - 1e-3)).all(-1).any(-1)
    assert inside.any() and np.sum(near.reshape(-1, 2).any(1) & ~near.reshape(-1, 2).all(1)) > 0   # pairs of one each
    if not np.isnan(bad):                                # (the network's ReLU makes a NaN zero)
        assert not np.isfinite(b[inside]).all(1).any()
    assert np.array_equal(a[~near].view(np.int32), b[~near].view(np.int32))


def test_field_forward_of_a_small_table_in_place(nsl, gpu):
    """Field.fwd of 16 levels of at most 2^10 entries, whose table the caches hold,
    takes no longer than nsl_field_fwd, which gathers in place (1.2 times with an
    encoding of its own)."""
    import torch
    spec = dataclasses.replace(W.C2_FIELD, log2_table=10, max_res=256)
    f = nsl.Field(spec)
    S = 600000
    P = _t(torch, gpu, params_for(spec, f.layout, seed=1, table_range=0.2)[0])
    X = torch.rand(S, 3, device=gpu)
    D = torch.nn.functional.normalize(torch.randn(S, 3, device=gpu), dim=1)
    ws = torch.empty(f.workspace_bytes(S), dtype=torch.uint8, device=gpu)
    sg, rgb = f.fwd(P, X, D, ws)
    direct = lambda: nsl._lib.nsl_field_fwd(f.handle, P.data_ptr(), X.data_ptr(), D.data_ptr(), S, sg.data_ptr(),
                                            rgb.data_ptr(), ws.data_ptr(), ws.numel(), nsl._stream())
    assert _shortest_ms(torch, lambda: f.fwd(P, X, D, ws)) < 1.1 * _shortest_ms(torch, direct)


@pytest.mark.parametrize("log2_table", [10, 16, 17])
def test_mixed_forward_around_the_level_walk(nsl, gpu, log2_table):
    """nsl_field_fwd_mixed of 16 levels whose FP16 table fits an L2 (2^10, 2^16
    entries) or does not (2^17): the bits of calls of fewer samples, and with 2^10
    entries 100003 samples take at most a third of the time they take with 2^19
    (0.26; level by level 0.41)."""
    import torch
    S = 100003
    X = torch.rand(S, 3, device=gpu)
    D = torch.nn.functional.normalize(torch.randn(S, 3, device=gpu), dim=1)

    def field(lg):
        f = nsl.Field(dataclasses.replace(W.C2_FIELD, log2_table=lg, max_res=2048 if lg > 10 else 256))
        return f, f.prepare_mixed(_t(torch, gpu, params_for(f.spec, f.layout, seed=1, table_range=0.2)[0]))

    f, sh = field(log2_table)
    sg, rgb = f.fwd_mixed(sh, X, D)
    for lo in range(0, S, 32000):
        a, b = f.fwd_mixed(sh, X[lo:lo + 32000].contiguous(), D[lo:lo + 32000].contiguous())
        assert torch.equal(sg[lo:lo + 32000], a) and torch.equal(rgb[lo:lo + 32000], b)
    if log2_table == 10:
        g, big = field(19)
        assert _shortest_ms(torch, lambda: f.fwd_mixed(sh, X, D)) < _shortest_ms(torch, lambda: g.fwd_mixed(big, X, D)) / 3


@pytest.mark.parametrize("spec", [W.C1_FIELD, MID_TABLES], ids=["in-lds", "fp16-in-lds"])
@pytest.mark.parametrize("S", [98303, 98304, 98305, 98816, 131071])
def test_encode_around_the_copy_to_lds(nsl, gpu, spec, S):
    """nsl_encode_fwd and nsl_encode_fwd_mixed around the sample count from which
    a small table is copied to LDS, and around its 512 samples a workgroup: the bits of
    calls of fewer samples, which read it from memory."""
    import torch
    f = nsl.Field(spec)
    P = _t(torch, gpu, params_for(spec, f.layout, seed=10, table_range=0.5)[0])
    sh = f.prepare_mixed(P)
    X = torch.rand(S, 3, device=gpu) * 1.04 - 0.02
    a, b = nsl.encode_fwd(f, P, X), nsl.encode_fwd_mixed(f, sh, X)
    for lo in range(0, S, 65000):
        x = X[lo:lo + 65000].contiguous()
        assert torch.equal(a[:, lo:lo + 65000], nsl.encode_fwd(f, P, x))
        assert torch.equal(b[:, lo:lo + 65000], nsl.encode_fwd_mixed(f, sh, x))
