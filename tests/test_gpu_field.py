"""GPU parity of the hash-encoded deformation fields (Sec. 3.3, App. B): dass_hash_field_fwd and
dass_hash_field_bwd against the float64 oracle, at the paper's table sizes and at small ones
that span dense and hashed levels, ragged query counts, queries outside the valid rows, and the
full-size field workload (200k Gaussians, one tenth dynamic)."""
import numpy as np
import pytest
import torch

import synth
from gpu_util import assert_grad_close, log
from oracle import hashfield as HF

pytestmark = pytest.mark.gpu

# (levels, features, log2_table, hidden, n_max): the N3DV dynamic and static fields (App. B),
# then small variants (dense-only, F = 1 and 8, hidden 32)
CONFIGS = {
    "n3dv_dyn": (16, 4, 16, 64, 2048),
    "n3dv_st": (16, 2, 14, 64, 2048),
    "meetroom_dyn": (16, 4, 15, 64, 2048),
    "dense_f1_h32": (6, 1, 18, 32, 48),
    "f8_h64": (8, 8, 12, 64, 256),
}


def dev(a, dtype=None):
    return torch.as_tensor(np.ascontiguousarray(a), device="cuda", dtype=dtype)


def make(name, seed=0):
    from paper_2411_14847_amd import HashField
    L, F, lt, hid, nmax = CONFIGS[name]
    p = synth.hash_field_params(seed, levels=L, features=F, log2_table=lt, hidden=hid, n_max=nmax)
    return p, HF.from_params(p), HashField.from_numpy(p, "cuda")


def clean_queries(f, mean, idx, margin=1e-4):
    """Drops queries with a hidden pre-activation within `margin` of zero: there the ReLU's
    branch is decided by rounding, and float32 and float64 may take different ones."""
    enc = HF.encode(f, HF.normalised(f, mean[:, idx]))
    pre = enc @ f.w1.T + f.b1
    keep = np.abs(pre).min(axis=1) > margin
    return idx[keep]


def run_case(name, n, m, seed, use_idx=True):
    from paper_2411_14847_amd import Context
    log(f"field parity {name} n={n} m={m} seed={seed} idx={use_idx}")
    p, f, fd = make(name, seed)
    mean, idx, ddp, ddr = synth.field_queries(seed + 100, n, m)
    if use_idx:
        idx = clean_queries(f, mean.astype(np.float64), idx)
    else:  # rows [0, m) of a mean array holding only unambiguous rows
        keep = clean_queries(f, mean.astype(np.float64), np.arange(n, dtype=np.int32))[:m]
        mean = np.ascontiguousarray(mean[:, keep])
        n = m = keep.size
        idx = np.arange(m, dtype=np.int32)
    m = idx.size
    ddp, ddr = ddp[:, :m], ddr[:, :m]
    ctx = Context(max_gaussians=max(n, 1), max_views=1, max_keys=1 << 10, max_tiles=16)
    dpos = torch.zeros(3, m, device="cuda")
    drot = torch.zeros(4, m, device="cuda")
    didx = dev(idx) if use_idx else None
    ctx.hash_field_fwd(fd, dev(mean), n, didx, m, dpos, drot)
    grads = fd.zeros_like()
    ctx.hash_field_bwd(fd, dev(mean), n, didx, m, dev(ddp), dev(ddr), grads)
    ctx.sync()
    mq = mean[:, idx].astype(np.float64)
    odp, odr = HF.field_fwd(f, mq)
    assert_grad_close("dpos", dpos.cpu().numpy(), odp)
    assert_grad_close("drot", drot.cpu().numpy(), odr)
    og = HF.field_bwd(f, mq, ddp, ddr)
    for k, t in zip(("table", "w1", "b1", "w2", "b2"), grads.arrays()):
        assert_grad_close(k, t.cpu().numpy(), og[k])


@pytest.mark.parametrize("name", list(CONFIGS))
def test_field_parity(name):
    run_case(name, 6000, 3001, 1)


def test_field_parity_rows_without_index():
    run_case("n3dv_st", 2500, 2500, 2, use_idx=False)


def test_field_invalid_rows_identity_and_no_gradient():
    from paper_2411_14847_amd import Context
    p, f, fd = make("f8_h64", 3)
    n = 500
    mean, idx, ddp, ddr = synth.field_queries(9, n, 200)
    idx = clean_queries(f, mean.astype(np.float64), idx)
    m = idx.size
    bad = idx.copy()
    bad[::7] = -1
    bad[3::7] = n          # == n: outside the valid rows
    ok = bad >= 0
    ok &= bad < n
    ctx = Context(max_gaussians=n, max_views=1, max_keys=1 << 10, max_tiles=16)
    dpos = torch.full((3, m), 7.0, device="cuda")
    drot = torch.full((4, m), 7.0, device="cuda")
    ctx.hash_field_fwd(fd, dev(mean), n, dev(bad), m, dpos, drot)
    grads = fd.zeros_like()
    ctx.hash_field_bwd(fd, dev(mean), n, dev(bad), m, dev(ddp[:, :m]), dev(ddr[:, :m]), grads)
    ctx.sync()
    dp, dr = dpos.cpu().numpy(), drot.cpu().numpy()
    assert np.all(dp[:, ~ok] == 0.0) and np.all(dr[0, ~ok] == 1.0) and np.all(dr[1:, ~ok] == 0.0)
    mq = mean[:, bad[ok]].astype(np.float64)
    odp, odr = HF.field_fwd(f, mq)
    assert_grad_close("dpos", dp[:, ok], odp)
    assert_grad_close("drot", dr[:, ok], odr)
    og = HF.field_bwd(f, mq, ddp[:, :m][:, ok], ddr[:, :m][:, ok])
    for k, t in zip(("table", "w1", "b1", "w2", "b2"), grads.arrays()):
        assert_grad_close(k, t.cpu().numpy(), og[k])


def test_field_identity_init_accumulation_and_errors():
    from paper_2411_14847_amd import Context, DassError, HashField, geometric_res
    ctx = Context(max_gaussians=1000, max_views=1, max_keys=1 << 10, max_tiles=16)
    fd = HashField.init(geometric_res(16, 2048, 16), 4, 16, 64, (-1.5,) * 3, (1.5,) * 3, "cuda", seed=4)
    mean, idx, ddp, ddr = synth.field_queries(4, 1000, 700)
    dpos = torch.zeros(3, 700, device="cuda")
    drot = torch.zeros(4, 700, device="cuda")
    ctx.hash_field_fwd(fd, dev(mean), 1000, dev(idx), 700, dpos, drot)
    ctx.sync()
    assert torch.all(dpos == 0) and torch.all(drot[0] == 1) and torch.all(drot[1:] == 0)
    # gradients accumulate: two identical backward calls give twice one
    g1, g2 = fd.zeros_like(), fd.zeros_like()
    ctx.hash_field_bwd(fd, dev(mean), 1000, dev(idx), 700, dev(ddp), dev(ddr), g1)
    ctx.hash_field_bwd(fd, dev(mean), 1000, dev(idx), 700, dev(ddp), dev(ddr), g2)
    ctx.hash_field_bwd(fd, dev(mean), 1000, dev(idx), 700, dev(ddp), dev(ddr), g2)
    ctx.sync()
    for a, b in zip(g1.arrays(), g2.arrays()):
        torch.testing.assert_close(b, 2 * a, rtol=1e-5, atol=1e-6 * float(a.abs().max()) + 1e-30)
    assert float(g1.b2.abs().max()) > 0 and float(g1.w2.abs().max()) > 0  # zero output layer: only w2, b2 move
    assert float(g1.w1.abs().max()) == 0 and float(g1.table.abs().max()) == 0
    # m = 0 is a no-op
    ctx.hash_field_fwd(fd, dev(mean), 1000, None, 0, dpos, drot)
    # invalid fields are refused before any launch
    for bad in (dict(res=[16] * 17), dict(features=3), dict(hidden=48), dict(log2_table=25),
                dict(aabb_max=(-2.0, 1.5, 1.5))):
        h = HashField(**{**fd.__dict__, **bad})
        with pytest.raises(DassError, match="DASS_E_INVALID"):
            ctx.hash_field_fwd(h, dev(mean), 1000, dev(idx), 700, dpos, drot)
    with pytest.raises(DassError, match="DASS_E_INVALID"):
        ctx.hash_field_fwd(fd, dev(mean), 1000, None, 1001, torch.zeros(3, 1001, device="cuda"),
                           torch.zeros(4, 1001, device="cuda"))


def test_field_fullsize_dynamic_and_static_groups():
    """The field workload of one training step: 200k Gaussians, 10% dynamic through the N3DV
    dynamic field, the rest through the static field, all outputs and gradients compared."""
    from paper_2411_14847_amd import Context
    n = 200_000
    rng = np.random.default_rng(11)
    mean = rng.uniform(-1.2, 1.2, size=(3, n)).astype(np.float32)
    dyn = np.sort(rng.choice(n, n // 10, replace=False)).astype(np.int32)
    st = np.setdiff1d(np.arange(n, dtype=np.int32), dyn).astype(np.int32)
    ctx = Context(max_gaussians=n, max_views=1, max_keys=1 << 10, max_tiles=16)
    for name, idx in (("n3dv_dyn", dyn), ("n3dv_st", st)):
        log(f"field fullsize {name} m={idx.size}")
        p, f, fd = make(name, 5)
        idx = clean_queries(f, mean.astype(np.float64), idx)
        m = idx.size
        ddp = rng.normal(size=(3, m)).astype(np.float32)
        ddr = rng.normal(size=(4, m)).astype(np.float32)
        dpos = torch.zeros(3, m, device="cuda")
        drot = torch.zeros(4, m, device="cuda")
        ctx.hash_field_fwd(fd, dev(mean), n, dev(idx), m, dpos, drot)
        grads = fd.zeros_like()
        ctx.hash_field_bwd(fd, dev(mean), n, dev(idx), m, dev(ddp), dev(ddr), grads)
        ctx.sync()
        mq = mean[:, idx].astype(np.float64)
        odp, odr = HF.field_fwd(f, mq)
        assert_grad_close("dpos", dpos.cpu().numpy(), odp)
        assert_grad_close("drot", drot.cpu().numpy(), odr)
        og = HF.field_bwd(f, mq, ddp, ddr)
        for k, t in zip(("table", "w1", "b1", "w2", "b2"), grads.arrays()):
            assert_grad_close(k, t.cpu().numpy(), og[k])


def test_fields_through_shift_match_oracle():
    """The shift of Sec. 3.3 driven by the two fields: offsets of the dynamic rows from H_dyn and
    of the static rows from H_st, laid out [dynamic | static] in one offset buffer, applied by
    shift_apply; then the adjoint of an upstream gradient back through shift_apply into both
    fields' parameters -- all against the oracle's composition of the same steps."""
    import oracle
    from paper_2411_14847_amd import Context
    scene, cams, _ = synth.single_view_scene(5, n=3000)
    n = scene.n
    rng = np.random.default_rng(21)
    dyn = np.sort(rng.choice(n, 300, replace=False)).astype(np.int32)
    st = np.setdiff1d(np.arange(n, dtype=np.int32), dyn).astype(np.int32)
    mean64 = scene.mean.astype(np.float64)
    parts = []
    from paper_2411_14847_amd import HashField
    box = (float(scene.mean.min()) - 0.05, float(scene.mean.max()) + 0.05)
    for name, idx, seed in (("n3dv_dyn", dyn, 6), ("n3dv_st", st, 7)):
        L, F, lt, hid, nmax = CONFIGS[name]
        p = synth.hash_field_params(seed, levels=L, features=F, log2_table=lt, hidden=hid, n_max=nmax, aabb=box)
        f = HF.from_params(p)
        parts.append((f, HashField.from_numpy(p, "cuda"), clean_queries(f, mean64, idx)))
    (fdy, fdy_d, dyn), (fst, fst_d, st) = parts
    nd, ns = dyn.size, st.size
    rows = np.concatenate([dyn, st]).astype(np.int32)
    from gpu_util import to_gpu
    g = to_gpu(scene)
    out = g.zeros_like()
    ctx = Context(max_gaussians=n, max_views=1, max_keys=1 << 12, max_tiles=64)
    dpos = torch.zeros(3, nd + ns, device="cuda")
    drot = torch.zeros(4, nd + ns, device="cuda")
    ctx.hash_field_fwd(fdy_d, g.mean, n, dev(dyn), nd, dpos, drot, col=0)
    ctx.hash_field_fwd(fst_d, g.mean, n, dev(st), ns, dpos, drot, col=nd)
    ctx.shift_fwd(g, out, dev(rows), dpos, drot)
    dmean = rng.normal(size=(3, n)).astype(np.float32)
    dquat = rng.normal(size=(4, n)).astype(np.float32)
    d_out = g.zeros_like()
    d_out.mean.copy_(dev(dmean))
    d_out.quat.copy_(dev(dquat))
    d_dpos = torch.zeros(3, nd + ns, device="cuda")
    d_drot = torch.zeros(4, nd + ns, device="cuda")
    ctx.shift_adjoint(g, dev(rows), drot, d_out, d_dpos, d_drot)
    gdy, gst = fdy_d.zeros_like(), fst_d.zeros_like()
    ctx.hash_field_bwd(fdy_d, g.mean, n, dev(dyn), nd, d_dpos, d_drot, gdy, col=0)
    ctx.hash_field_bwd(fst_d, g.mean, n, dev(st), ns, d_dpos, d_drot, gst, col=nd)
    ctx.sync()
    # oracle composition
    a_dp, a_dr = HF.field_fwd(fdy, mean64[:, dyn])
    b_dp, b_dr = HF.field_fwd(fst, mean64[:, st])
    o_dp, o_dr = np.concatenate([a_dp, b_dp], 1), np.concatenate([a_dr, b_dr], 1)
    om, oq = oracle.shift_fwd(scene, rows, o_dp, o_dr)
    assert_grad_close("mean", out.mean.cpu().numpy(), om)
    assert_grad_close("quat", out.quat.cpu().numpy(), oq)
    oddp, oddr = oracle.shift_adj(scene, rows, o_dr, dmean, dquat)
    assert_grad_close("d_dpos", d_dpos.cpu().numpy(), oddp)
    assert_grad_close("d_drot", d_drot.cpu().numpy(), oddr)
    for f, gd, sl in ((fdy, gdy, slice(0, nd)), (fst, gst, slice(nd, nd + ns))):
        idx = dyn if sl.start == 0 else st
        og = HF.field_bwd(f, mean64[:, idx], oddp[:, sl], oddr[:, sl])
        for k, t in zip(("table", "w1", "b1", "w2", "b2"), gd.arrays()):
            assert_grad_close(k, t.cpu().numpy(), og[k])


@pytest.mark.parametrize("use_graph", [False, True])
def test_streaming_with_hash_fields(use_graph):
    """The streaming driver with the H_dyn / H_st shift: the loss falls within each timestep and
    densification and erasure behave as with direct offsets."""
    from paper_2411_14847_amd import Context, GaussianBuffers
    from paper_2411_14847_amd.streaming import StreamConfig, Trainer
    scene, _, _ = synth.single_view_scene(0, n=600)
    cams = synth.streaming_rig(64, 64)[:4]
    cfg = StreamConfig(iters=25, k_append=80, erase_every=2, use_graph=use_graph, shift="hash",
                       field_dyn=(8, 4, 12, 64, 4, 64), field_st=(8, 2, 10, 32, 4, 32))
    cap = scene.n + 2 * cfg.k_append
    g = GaussianBuffers.from_arrays(scene.mean, scene.quat, scene.log_scale, scene.logit, scene.sh, 0, capacity=cap)
    gt = g.clone()
    ctx = Context(max_gaussians=cap, max_views=len(cams), max_keys=cap * len(cams) * 32, max_tiles=4 * 16)
    tr = Trainer(ctx, g, cams, max_dynamic=scene.n // 10, cfg=cfg)
    gt_ctx = Context(max_gaussians=cap, max_views=len(cams), max_keys=cap * len(cams) * 32, max_tiles=4 * 16)
    ns = []
    for t in range(1, 4):
        m = synth.timestep_motion(0, t, scene.n)
        gt_out = gt.zeros_like()
        gt_ctx.shift_fwd(gt, gt_out, dev(m.dynamic), dev(m.dpos), dev(m.dquat))
        gt.mean.copy_(gt_out.mean); gt.quat.copy_(gt_out.quat)
        targets = [o.rgb.clone() for o in gt_ctx.render_fwd(gt, cams, cfg.bg)]
        st = tr.timestep(t, dev(m.dynamic), targets)
        log(f"  t={t} loss {st['loss_first']:.5f} -> {st['loss_last']:.5f}, appended {st['appended']}, n {st['n']}")
        assert st["loss_last"] < st["loss_first"]
        ns.append(st["n"])
    ctx.sync()
    assert ns[0] == scene.n + 80 and ns[1] == scene.n + 80 and ns[2] == scene.n + 160


@pytest.mark.parametrize("L,F,lt,nmax,m", [
    (4, 4, 12, 256, 1),        # one slice a level, one query
    (5, 4, 13, 256, 1023),     # hashed levels of two slices, the second ragged; queries below a workgroup's
    (6, 2, 14, 512, 2047),     # a query part takes at least 1024: still one part
    (6, 2, 14, 512, 2049),     # two parts, partial slices added
    (16, 1, 15, 2048, 5000),   # two slices a level, as many parts as the queries give
    (8, 8, 16, 1024, 4500),    # 26 slices a hashed level, parts for the dense ones only
    (8, 8, 18, 1024, 2500),    # more slices than workgroups of one round
])
def test_field_table_gradient_at_slice_and_part_edges(monkeypatch, L, F, lt, nmax, m):
    monkeypatch.setitem(CONFIGS, "edge", (L, F, lt, 64, nmax))
    run_case("edge", 2 * m + 10, m, 5)


@pytest.mark.parametrize("offset", [0, 2])
def test_field_of_two_features_reads_row_pairs(offset):
    """F = 2: two neighbouring rows are one 16-byte load, from a table that starts on 8 bytes only; the last
    row of a level, dense and hashed, included (positions at the box's upper corner).  Against the oracle."""
    from paper_2411_14847_amd import Context
    p = synth.hash_field_params(21, levels=6, features=2, log2_table=12, hidden=32, n_max=256)
    f = HF.from_params(p)
    from paper_2411_14847_amd import HashField
    fd = HashField.from_numpy(p, "cuda")
    buf = torch.zeros(fd.table.numel() + 4, device="cuda")
    buf[offset:offset + fd.table.numel()] = fd.table.reshape(-1)
    fd.table = buf[offset:offset + fd.table.numel()].view(fd.table.shape)
    mean, idx, _, _ = synth.field_queries(22, 900, 500)
    mean[:, idx[:40]] = np.asarray(f.aabb_max if hasattr(f, "aabb_max") else p.aabb_max, np.float32)[:, None]
    mean[:, idx[40:80]] = np.asarray(p.aabb_min, np.float32)[:, None]
    ctx = Context(max_gaussians=900, max_views=1, max_keys=1 << 10, max_tiles=16)
    dpos, drot = torch.zeros(3, 500, device="cuda"), torch.zeros(4, 500, device="cuda")
    log(f"field row pairs, table {offset} floats off")
    ctx.hash_field_fwd(fd, dev(mean), 900, dev(idx), 500, dpos, drot)
    ctx.sync()
    odp, odr = HF.field_fwd(f, mean[:, idx].astype(np.float64))
    assert_grad_close("dpos", dpos.cpu().numpy(), odp)
    assert_grad_close("drot", drot.cpu().numpy(), odr)
