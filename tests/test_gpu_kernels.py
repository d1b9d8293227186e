"""Kernel variants and dispatch branches at the sizes where they can go
wrong, against the FP64 oracle."""
import ctypes

import numpy as np
import pytest
import torch

import oracle
from paper_2606_08469_amd import binding, synth

from _gpu import rel_l2, report, to_np
from _tiny import tiny_problem

pytestmark = pytest.mark.gpu


def random_mlp(widths, dtype, seed, off=0):
    """FP32 weights, and a device MLP whose weights start `off` elements into
    their buffers (off = 1: aligned for single elements only)."""
    g = np.random.default_rng(seed)
    W = [(g.uniform(-1, 1, (o, i)) * np.sqrt(6.0 / (i + o))).astype(np.float32) for i, o in zip(widths, widths[1:])]
    b = [(0.1 * g.normal(size=o)).astype(np.float32) for o in widths[1:]]
    dev = []
    for w in W:
        buf = torch.zeros(w.size + off, dtype=dtype, device="cuda")
        buf[off:] = torch.from_numpy(w.reshape(-1)).to(dtype)
        dev.append(buf[off:].view(w.shape))
    ref = [to_np(w).astype(np.float32) for w in dev]  # the rounded weights
    return binding.MLP(dev, [torch.from_numpy(v).cuda() for v in b]), oracle.MLP(ref, b)


@pytest.mark.parametrize("widths", [(20, 64, 3), (64, 64, 64, 64, 3), (76, 128, 128, 3), (128, 128, 128, 128, 128, 3)])
@pytest.mark.parametrize("dtype", [torch.float16, torch.bfloat16, torch.float32])
@pytest.mark.parametrize("B,off", [(1, 0), (15, 1), (33, 0), (64, 0), (65, 1), (130, 0), (8 * 256 * 64 + 17, 0)])
def test_decoder_shapes(widths, dtype, B, off):
    """One to four input chunks, ragged row counts, weights aligned for whole
    fragments or not, weights in LDS or (FP32, four 128-wide layers) not.
    FP32: products and sums of at most 128 terms per layer, 1e-5. 16 bit:
    each layer rounds its activations to 2^-11 (2^-8 for BF16) relative, at
    most four roundings deep: 4 * 2^-8 < 0.02 of a row's scale."""
    if B > 1000 and (dtype == torch.bfloat16 or widths[0] == 20):
        pytest.skip("the persistent loop is covered by the other shapes")
    print(f"[case] decoder {widths} {dtype} B={B} off={off}", flush=True)
    mlp, omlp = random_mlp(widths, dtype, 7, off)
    h = (0.5 * torch.randn(B, widths[0], generator=torch.Generator().manual_seed(B))).to(dtype).cuda()
    rgb = to_np(binding.mlp_fwd(mlp, h))
    rows = np.arange(B) if B < 1000 else np.concatenate([np.arange(64), np.arange(B - 200, B)])
    want = oracle.mlp_fwd(omlp, to_np(h)[rows].astype(np.float64))
    rms = float(np.sqrt(np.mean(want ** 2)))
    worst = float(np.max(np.abs(rgb[rows] - want) / (np.abs(want) + rms)))
    report(f"decoder {widths} {dtype} B={B}", worst=worst)
    assert worst <= (1e-5 if dtype == torch.float32 else 0.02)


def small_paper_model(dtype, widths):
    """Four levels of vertex maps over a random tree, with a predictor of one
    or two hidden layers and a decoder that reads 4 attributes."""
    g = np.random.default_rng(11)
    s = (g.uniform(0, 1, (4000, 3)) ** 1.5).astype(np.float32)
    nodes, lo = binding.build_octree(s, 3, 8)
    res, C = [8, 8, 4, 2], 4
    feat = [g.normal(0, 0.1, (int(n), r + 1, r + 1, C)).astype(np.float32) for n, r in zip(np.diff(lo), res)]
    W, b = [], []
    for i, o in ((20, 64), (64, 64), (64, 3)):
        W.append((g.uniform(-1, 1, (o, i)) * np.sqrt(6.0 / (i + o))).astype(np.float32))
        b.append((0.1 * g.normal(size=o)).astype(np.float32))
    cfg = synth.CONFIGS[6]
    disp = synth.init_disparity(cfg, log2_T=10, table_scale=0.5, d0=1.5, widths=widths)
    for v in disp["b"][:-1]:
        v[:] = 0.1 * g.normal(size=v.shape)
    model = binding.OctaOctree(nodes, lo, res, C, feat, W, b, dtype=dtype, interp=binding.INTERP_PAPER, disparity=disp)
    od = oracle.Disparity(disp["res"], synth.HASH_F, disp["log2_T"], disp["tables"], disp["W"], disp["b"])
    return model, oracle.Tree(nodes, lo, res, C, feat, interp=binding.INTERP_PAPER, disp=od), oracle.MLP(W, b)


@pytest.mark.parametrize("dtype", [torch.float32, torch.float16])
@pytest.mark.parametrize("widths", [(64,), (64, 64)])
@pytest.mark.parametrize("B", [1, 63, 65, 1000, (1 << 20) + 65])
def test_shifted_query_routes(dtype, widths, B):
    """The shifted query with a workspace (three kernels, two passes above
    2^20 queries), without one (predictor, then the fused kernel) and the
    encode + decode pair: the first two agree bit for bit, and all with the
    oracle at the bars of the shifted query (1e-5 in FP32, 1e-2 in FP16)."""
    model, otree, omlp = small_paper_model(dtype, widths)
    g = np.random.default_rng(B)
    x = torch.from_numpy(g.uniform(-0.02, 1.02, (B, 3)).astype(np.float32)).cuda()
    d = torch.from_numpy(g.normal(size=(B, 3)).astype(np.float32)).cuda()
    attr = torch.from_numpy(g.normal(size=(B, 4)).astype(np.float32)).cuda()
    print(f"[case] shifted query {dtype} {widths} B={B}", flush=True)
    split = model(x, d, attr)
    fused = torch.full((B, 3), 7.0, device="cuda")
    ts, ms = model.tree.struct(model.work_feat), model.mlp.struct(model.work_W)
    p = lambda t: ctypes.c_void_p(t.data_ptr())
    assert binding.lib().oo_query_fwd(ctypes.byref(ts), ctypes.byref(ms), p(x), p(d), p(attr), B, p(fused),
                                      ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)) == 0
    assert torch.equal(split, fused)
    rows = np.unique(np.concatenate([np.arange(min(B, 200)), np.arange(max(0, B - 200), B)]))
    want = oracle.query_fwd(otree, omlp, x.cpu().numpy()[rows], d.cpu().numpy()[rows], attr=attr.cpu().numpy()[rows])
    err = rel_l2(to_np(split)[rows], want)
    h, _ = binding.encode_query(model.tree, x, d, with_idx=False, feat=model.work_feat)
    oh = oracle.encode(otree, x.cpu().numpy()[rows], d.cpu().numpy()[rows])[0]
    herr = rel_l2(to_np(h)[rows], oh)
    report(f"shifted query {dtype} {widths} B={B}", rgb=err, h=herr)
    tol = 1e-5 if dtype == torch.float32 else 1e-2
    assert err <= tol and herr <= tol


def test_shifted_query_refuses_short_workspace():
    model, _, _ = small_paper_model(torch.float32, (64,))
    x = torch.rand(100, 3, device="cuda")
    attr, rgb = torch.rand(100, 4, device="cuda"), torch.full((100, 3), 7.0, device="cuda")
    ts, ms = model.tree.struct(), model.mlp.struct()
    n = ctypes.c_size_t(0)
    L = binding.lib()
    assert L.oo_query_workspace_bytes(ctypes.byref(ts), ctypes.byref(ms), 100, ctypes.byref(n)) == 0 and n.value > 0
    ws = torch.empty(n.value, dtype=torch.uint8, device="cuda")
    p = lambda t: ctypes.c_void_p(t.data_ptr())
    for w, size in ((p(ws), n.value - 1), (None, n.value)):
        assert L.oo_query_fwd_ws(ctypes.byref(ts), ctypes.byref(ms), p(x), p(x), p(attr), 100, p(rgb), w, size, None) == -1
    torch.cuda.synchronize()
    assert torch.all(rgb == 7.0)


@pytest.mark.parametrize("widths,n_attr", [((64,), 0), ((64, 64, 64, 64), 112), ((128,), 4), ((128, 128), 8),
                                           ((128, 128), 112), ((128, 128, 128), 48), ((128,) * 4, 32),
                                           ((128,) * 4, 72), ((128,) * 4, 112)])
@pytest.mark.parametrize("dtype", [torch.float16, torch.bfloat16])
@pytest.mark.parametrize("B", [1, 17, 129, 700])
def test_decoder_backward_shapes(widths, n_attr, dtype, B):
    """Every workgroup shape of the 16-bit backward: no to three
    hidden-to-hidden layers, four or eight waves, exchange buffers for all or
    a share of the waves, and the widest decoder, which runs the kernel with
    weights in L2; batches that end inside a tile and inside a wave's 16
    queries. Loss and weight gradients against plain FP64 torch that rounds
    inputs, activations, seeds and deltas to 16 bits where the kernel does.
    What is left is FP32 sums that round to the other 16-bit neighbour, now
    and then, in up to five layers: 10 units of 2^-11 (2^-8 for BF16)."""
    tree, mlp, bt = tiny_problem(seed=5, widths=widths, B=max(B, 2), N=0, n_attr=n_attr, bias_scale=0.1)
    bt = {k: (v[:B] if isinstance(v, np.ndarray) else v) for k, v in bt.items()}
    bt["target_override"] = np.random.default_rng(1).uniform(0, 1, (B, 3)).astype(np.float32)
    print(f"[case] backward {widths} E={n_attr} {dtype} B={B}", flush=True)
    model = binding.OctaOctree(tree.nodes, tree.level_offset, tree.res, tree.C, tree.feat, mlp.W, mlp.b, dtype=dtype)
    dev = binding.device_batch(bt)
    loss = model.residual(dev)
    loss.backward()
    h, _ = binding.encode_query(model.tree, dev["x"], dev["dir"], dtype, feat=model.work_feat)
    r16 = lambda t: t.to(dtype).double()
    a = [h.double() if n_attr == 0 else torch.cat([h.double(), r16(dev["attr"])], 1)]
    W = [w.double() for w in model.work_W]
    b = [v.detach().double() for v in model.b]
    z = []
    for i in range(len(W) - 1):
        z.append(a[-1] @ W[i].T + b[i])
        a.append(r16(z[i].relu()))
    res = a[-1] @ W[-1].T + b[-1] - dev["target_override"].double()
    want = (res * res).sum() / (3 * B)
    bar = 10 * (2.0 ** -11 if dtype == torch.float16 else 2.0 ** -8)

    def error(open_):
        d = r16(2 * res)
        worst = abs(float(loss.detach()) / float(want) - 1)
        for i in reversed(range(len(W))):
            for got, ref in ((model.W[i].grad, d.T @ a[i] / (3 * B)), (model.b[i].grad, d.sum(0) / (3 * B))):
                if ref.norm() > 0:
                    worst = max(worst, float((got.double() - ref).norm() / ref.norm()))
            if i:
                d = r16((d @ W[i]) * open_[i - 1])
        dh = (d @ W[0])[:, :tree.n_levels * tree.C] / (3 * B)
        # a level's map entries collect dh with weights that sum to one per query
        for l, f in enumerate(model.feat):
            has = torch.from_numpy(oracle.descend(tree, bt["x"])[:, l] >= 0).cuda()
            ref = (dh[:, l * tree.C:(l + 1) * tree.C] * has[:, None]).sum(0)
            got = f.grad.double().sum((0, 1, 2))
            scale = (dh[:, l * tree.C:(l + 1) * tree.C] * has[:, None]).abs().sum(0).norm()
            if scale > 0:
                worst = max(worst, float((got - ref).norm() / scale))
        return worst

    # A unit whose sum lies nearer to zero than one input's rounding to its
    # other neighbour moves it has no one derivative: the kernel may take
    # either side, and the reference goes along with it, the nearest first.
    open_ = [x > 0 for x in a[1:]]
    worst = error(open_)
    if worst > bar:
        near = [(float(z[i][q, n].abs()), i, q, n) for i in range(len(z)) for q, n in
                (z[i].abs() < bar / 10 * (a[i][:, None] * W[i]).abs().amax(-1)).nonzero().tolist()]
        for _, i, q, n in sorted(near)[:64]:
            open_[i][q, n] ^= True
            e = error(open_)
            if e < worst:
                worst = e
            else:
                open_[i][q, n] ^= True
    report(f"backward {widths} E={n_attr} {dtype} B={B}", worst=worst)
    assert worst <= bar


@pytest.mark.parametrize("D", [4, 5, 7])
@pytest.mark.parametrize("B,N", [(1, 0), (262143, 0), (262144, 0), (270001, 0), (40000, 6), (5000, 60)])
def test_shifted_residual_query_order(D, B, N):
    """The finer query order of the shifted residual (tree depths where it has
    no, one and two levels to add; batches around the smallest it takes; runs
    that end early; more buckets in a run
    than have ranks of their own, since the points fill the cube): a query's
    result does not depend on where it is evaluated, so permuting the batch
    permutes every output, bit for bit, and the corner nodes."""
    res = (8, 8, 4, 4, 2, 2, 2, 2)[:D + 1]
    tree, _, _ = tiny_problem(seed=3, D=D, res=res, B=2, N=0)
    g = np.random.default_rng(11)
    bt = tiny_problem(seed=4, D=D, res=res, B=max(B, 2), N=N, widths=(64,), n_attr=0)[2]
    bt = {k: (v[:B] if isinstance(v, np.ndarray) else v) for k, v in bt.items()}
    bt["x"] = g.uniform(0, 1, (B, 3)).astype(np.float32)
    if N == 0:
        bt["target_override"] = g.uniform(0, 1, (B, 3)).astype(np.float32)
    feat = [g.normal(0, 0.1, (len(f), r + 1, r + 1, 4)).astype(np.float32) for f, r in zip(tree.feat, res)]
    W = [g.uniform(-0.3, 0.3, s).astype(np.float32) for s in ((64, 4 * (D + 1)), (3, 64))]
    b = [np.zeros(s, np.float32) for s in (64, 3)]
    disp = synth.init_disparity(synth.CONFIGS[6], log2_T=10, table_scale=0.5, d0=1.5)
    model = binding.OctaOctree(tree.nodes, tree.level_offset, list(res), 4, feat, W, b, dtype=torch.float16,
                               interp=binding.INTERP_PAPER, disparity=disp)
    print(f"[case] query order D={D} B={B} N={N}", flush=True)

    def run(batch):
        dev = binding.device_batch(batch)
        ws = model.workspace(dev)
        lhs, rhs, resid, loss = binding.residual_fwd(model.tree, model.mlp, dev, ws, feat=model.work_feat, W=model.work_W)
        idx = binding.residual_node_indices(model.tree, model.mlp, dev, ws, feat=model.work_feat, W=model.work_W)
        return [to_np(t) for t in (lhs, rhs, resid, idx)]

    p = g.permutation(B)
    moved = {k: (v[p] if isinstance(v, np.ndarray) else v) for k, v in bt.items()}
    for name, u, v in zip(("lhs", "rhs", "resid", "idx"), run(bt), run(moved)):
        assert np.array_equal(u[p], v), name


@pytest.mark.parametrize("levels,C,n_attr", [(1, 4, 0), (4, 4, 4), (4, 8, 0), (4, 8, 28), (4, 8, 96), (3, 8, 4)])
@pytest.mark.parametrize("dtype", [torch.float32, torch.float16, torch.bfloat16])
@pytest.mark.parametrize("B", [1, 65, 4099, 150001])
def test_streamed_query(levels, C, n_attr, dtype, B):
    """64-wide decoders, whose first layer takes the inputs in chunks of 32 as
    they are gathered: inputs that end with a chunk, within one and in the
    surface attributes, up to the most; single queries up to more than eight
    tiles per compute unit. The encoding followed by the standalone decoder
    adds the same products in the same order: equal to the bit."""
    res = (8, 4, 4, 2)[:levels]
    tree, mlp, _ = tiny_problem(seed=6, D=levels - 1, res=res, C=C, B=2, N=0, n_attr=n_attr, bias_scale=0.1)
    model = binding.OctaOctree(tree.nodes, tree.level_offset, list(res), C, tree.feat, mlp.W, mlp.b, dtype=dtype)
    g = np.random.default_rng(B)
    t = lambda *s: torch.from_numpy(g.uniform(0, 1, s).astype(np.float32)).cuda()
    x, d, attr = t(B, 3), t(B, 3) - 0.5, t(B, n_attr) if n_attr else None
    print(f"[case] streamed query L={levels} C={C} E={n_attr} {dtype} B={B}", flush=True)
    rgb = model(x, d, attr) if n_attr else model(x, d)
    h, _ = binding.encode_query(model.tree, x, d, dtype, feat=model.work_feat)
    if n_attr:
        h = torch.cat([h, attr.to(dtype)], 1)
    assert torch.equal(rgb, binding.mlp_fwd(model.mlp, h.contiguous(), W=model.work_W))


@pytest.mark.parametrize("B", [1, 1025, 65600, 66000, 200000, 262145])
def test_residual_query_order(B):
    """The bucketed order over one chunk of queries, a few, one more than a
    quarter of the most and all of them: a query's result does not depend on
    where it is evaluated, so permuting the batch permutes every output and
    the node indices, bit for bit."""
    tree, mlp, _ = tiny_problem(seed=8, D=4, res=(8, 8, 4, 4, 2), B=2, N=0)
    g = np.random.default_rng(12)
    f32 = lambda *s: g.uniform(-1, 1, s).astype(np.float32)
    bt = dict(x=0.5 + 0.5 * f32(B, 3), dir=f32(B, 3), n=f32(B, 3), wo=f32(B, 3), albedo=f32(B, 3), rough=f32(B),
              Le=f32(B, 3), N=0, F0=0.04, loss_kind=0, eps=1e-2, grad_through_rhs=0, target_override=f32(B, 3),
              wi=None, pdf=None, x2=None, dir2=None)
    model = binding.OctaOctree(tree.nodes, tree.level_offset, tree.res, 4, tree.feat, mlp.W, mlp.b)
    print(f"[case] residual order B={B}", flush=True)

    def run(batch):
        dev = binding.device_batch(batch)
        ws = model.workspace(dev)
        out = binding.residual_fwd(model.tree, model.mlp, dev, ws, feat=model.work_feat, W=model.work_W)
        idx = binding.residual_node_indices(model.tree, model.mlp, dev, ws, feat=model.work_feat, W=model.work_W)
        return [to_np(t) for t in (out[0], out[2], idx)]

    p = g.permutation(B)
    moved = {k: (v[p] if isinstance(v, np.ndarray) else v) for k, v in bt.items()}
    base = run(bt)
    for name, u, v in zip(("lhs", "resid", "idx"), base, run(moved)):
        assert np.array_equal(u[p], v), name
    assert np.array_equal(base[2], oracle.descend(tree, bt["x"]))


@pytest.mark.parametrize("res,B,spread", [((8, 8, 8), 131071, 1.0), ((8, 8, 8), 131072, 1.0), ((8, 16, 8, 8), 140001, 0.1),
                                          ((32, 32, 32), 150001, 0.03), ((8, 32, 16, 2), 262145, 0.3)])
@pytest.mark.parametrize("dtype", [torch.float32, torch.float16])
def test_coarse_scatter(res, B, spread, dtype):
    """Feature gradients of a batch large enough for the scatter that adds up
    shared footprints first, against the same points in batches too small for
    it (whose gradients add up, weighted by their points): the least number of
    points and one less, nodes that few points share, runs over more
    footprints than have counters, several runs per level. The same products
    in another order: 2^-24 times the terms of a sum, at most 2^16 a texel
    and mostly of both signs, so 2^-24 * 2^8 * 4 of the gradient's norm."""
    tree, mlp, _ = tiny_problem(seed=9, D=len(res) - 1, res=res, C=8, B=2, N=0)
    g = np.random.default_rng(13)
    u = lambda *s: g.uniform(0, 1, s).astype(np.float32)
    x = u(B, 3) * np.where(u(B, 1) < spread, 1.0, 0.2).astype(np.float32)
    bt = dict(x=x, dir=u(B, 3) - np.float32(0.5), n=u(B, 3), wo=u(B, 3), albedo=u(B, 3), rough=u(B), Le=u(B, 3), N=0,
              F0=0.04, loss_kind=0, eps=1e-2, grad_through_rhs=0, target_override=u(B, 3), wi=None, pdf=None, x2=None,
              dir2=None)
    model = binding.OctaOctree(tree.nodes, tree.level_offset, list(res), 8, tree.feat, mlp.W, mlp.b, dtype=dtype)
    print(f"[case] coarse scatter res={res} B={B} spread={spread} {dtype}", flush=True)

    def grads(lo, hi):
        part = {k: (v[lo:hi] if isinstance(v, np.ndarray) else v) for k, v in bt.items()}
        for f in model.feat:
            f.grad = None
        model.residual(binding.device_batch(part)).backward()
        return [f.grad.double() * (hi - lo) for f in model.feat]

    whole = grads(0, B)
    want = [torch.zeros_like(w) for w in whole]
    for lo in range(0, B, 30000):
        for w, p in zip(want, grads(lo, min(lo + 30000, B))):
            w += p
    for l, (a, b) in enumerate(zip(whole, want)):
        assert b.norm() > 0
        assert float((a - b).norm() / b.norm()) <= 2.0 ** -14, l


@pytest.mark.parametrize("dtype", [torch.float32, torch.float16])
@pytest.mark.parametrize("B", [1, 16384, 16385])
def test_residual_query_launches(dtype, B):
    """Backward's and secondary queries in one launch (up to 2^15 queries)
    and in two: what a query gives does not depend on it. LHS radiance equal
    to the plain query's to the bit, node indices to the oracle's."""
    tree, mlp, bt = tiny_problem(seed=10, D=3, res=(8, 4, 4, 2), B=max(B, 2), N=1)
    bt = {k: (v[:B] if isinstance(v, np.ndarray) else v) for k, v in bt.items()}
    model = binding.OctaOctree(tree.nodes, tree.level_offset, tree.res, 4, tree.feat, mlp.W, mlp.b, dtype=dtype)
    dev = binding.device_batch(bt)
    print(f"[case] residual launches B={B} {dtype}", flush=True)
    ws = model.workspace(dev)
    lhs = binding.residual_fwd(model.tree, model.mlp, dev, ws, feat=model.work_feat, W=model.work_W)[0]
    idx = binding.residual_node_indices(model.tree, model.mlp, dev, ws, feat=model.work_feat, W=model.work_W)
    assert torch.equal(lhs, model(dev["x"], dev["dir"]))
    assert np.array_equal(to_np(idx), oracle.descend(tree, bt["x"]))
