"""The residual forward's query launches, one or two of them."""
import numpy as np
import pytest
import torch

import oracle
from paper_2606_08469_amd import binding

from test_gpu_backward_chunks import paper_problem, points

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", [torch.float32, torch.float16])
@pytest.mark.parametrize("interp", [binding.INTERP_NODE_BILINEAR, binding.INTERP_PAPER])
@pytest.mark.parametrize("B,N", [(16384, 1), (16385, 1), (8193, 3), (100003, 4), (262081, 3), (262144, 1), (200001, 5)])
def test_two_query_launches(dtype, interp, B, N):
    """The backward's and the secondary queries in one launch (up to 100,003
    points here) and in two (the others: equally many rounds, or enough of
    them): what a query gives does not depend on it. LHS radiance
    equal to the plain query's to the bit, the targets to those of the first
    points in a batch of their own (one launch), node indices to the
    oracle's."""
    tree, feat, mlp, bt = paper_problem(B, N, 0, (64, 64), 18)
    if interp == binding.INTERP_NODE_BILINEAR:
        feat = [np.ascontiguousarray(f[:, :r, :r]) for f, r in zip(feat, tree.res)]
    bt["x"] = points(B)
    model = binding.OctaOctree(tree.nodes, tree.level_offset, list(tree.res), 4, feat, mlp.W, mlp.b, dtype=dtype,
                               interp=interp)
    dev = binding.device_batch(bt)
    print(f"[case] query launches B={B} N={N} {dtype} interp={interp}", flush=True)
    ws = model.workspace(dev)
    lhs, rhs = binding.residual_fwd(model.tree, model.mlp, dev, ws, feat=model.work_feat, W=model.work_W)[:2]
    assert torch.equal(lhs, model(dev["x"], dev["dir"]))
    few = {k: (v[:1000] if isinstance(v, np.ndarray) else v) for k, v in bt.items()}
    few = binding.device_batch(few)
    ws2 = model.new_workspace(few)
    rhs2 = binding.residual_fwd(model.tree, model.mlp, few, ws2, feat=model.work_feat, W=model.work_W)[1]
    assert torch.equal(rhs[:1000], rhs2)
    idx = binding.residual_node_indices(model.tree, model.mlp, dev, ws, feat=model.work_feat, W=model.work_W)
    if interp == binding.INTERP_NODE_BILINEAR:
        assert np.array_equal(idx.cpu().numpy(), oracle.descend(tree, bt["x"]))
