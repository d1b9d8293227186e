"""Queries whose radiance goes where their positions or directions were, and
queries without memory for a workspace."""
import ctypes

import pytest
import torch

from paper_2606_08469_amd import binding

from test_gpu_kernels import small_paper_model
from test_gpu_backward_chunks import paper_problem

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("predictor", [None, (64,), (64, 64)])
@pytest.mark.parametrize("dtype", [torch.float32, torch.float16, torch.bfloat16])
@pytest.mark.parametrize("B", [1, 65, 70001])
def test_radiance_over_an_input(predictor, dtype, B):
    """oo_query_fwd (no workspace) with rgb_out the array of the positions, and
    of the directions: the radiance of a call with an array of its own, bit for
    bit, with a disparity predictor and without."""
    if predictor:
        model, _, _ = small_paper_model(dtype, predictor)
    else:
        tree, feat, mlp, _ = paper_problem(2, 0, 4, (64, 64), 19)
        model = binding.OctaOctree(tree.nodes, tree.level_offset, list(tree.res), 4, feat, mlp.W, mlp.b, dtype=dtype,
                                   interp=binding.INTERP_PAPER)
    g = torch.Generator().manual_seed(B)
    x, d = torch.rand(B, 3, generator=g).cuda(), torch.randn(B, 3, generator=g).cuda()
    attr = torch.randn(B, 4, generator=g).cuda()
    print(f"[case] radiance over an input {predictor} {dtype} B={B}", flush=True)
    ts, ms = model.tree.struct(model.work_feat), model.mlp.struct(model.work_W)
    p = lambda t: ctypes.c_void_p(t.data_ptr())

    def query(x, d, out):
        assert binding.lib().oo_query_fwd(ctypes.byref(ts), ctypes.byref(ms), p(x), p(d), p(attr), B, p(out),
                                          ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)) == 0
        return out

    want = query(x, d, torch.empty_like(x))
    assert torch.equal(model(x, d, attr), want)
    over_x, over_d = x.clone(), d.clone()
    assert torch.equal(query(over_x, d, over_x), want)
    assert torch.equal(query(x, over_d, over_d), want)
    for over, at in ((x.clone(), 0), (d.clone(), 1)):  # the binding's route, with a workspace
        ins = [over if at == i else t for i, t in enumerate((x, d))]
        assert torch.equal(binding.query_fwd(model.tree, model.mlp, *ins, feat=model.work_feat, W=model.work_W,
                                             out=over, attr=attr), want)


def test_query_without_room_for_a_workspace(monkeypatch):
    """binding.query_fwd where the device has no memory left for the workspace
    of a model with a predictor: the call that needs none, same bits."""
    model, _, _ = small_paper_model(torch.float16, (64, 64))
    x, d, attr = torch.rand(999, 3).cuda(), torch.randn(999, 3).cuda(), torch.randn(999, 4).cuda()
    out = torch.empty(999, 3, device="cuda")
    want = model(x, d, attr).clone()
    empty = torch.empty

    def no_room(*size, **kw):
        if kw.get("dtype") == torch.uint8:
            raise torch.OutOfMemoryError("no room")
        return empty(*size, **kw)

    monkeypatch.setattr(torch, "empty", no_room)
    print("[case] query without room for a workspace", flush=True)
    got = binding.query_fwd(model.tree, model.mlp, x, d, feat=model.work_feat, W=model.work_W, out=out, attr=attr)
    assert got is out and torch.equal(got, want)
