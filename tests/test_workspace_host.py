"""Size of the residual step's workspace (no GPU needed)."""
import ctypes as C

import pytest

from paper_2606_08469_amd import binding
from test_abi_host import L, _mlp, _tree  # noqa: F401


@pytest.mark.parametrize("H,hidden", [(64, 1), (64, 4), (128, 2), (128, 4)])
@pytest.mark.parametrize("E", [0, 16, 72, 104])
@pytest.mark.parametrize("interp", [0, 1])
@pytest.mark.parametrize("N,full", [(0, 0), (1, 0), (3, 0), (32, 0), (3, 1)])
@pytest.mark.parametrize("dtype", [binding.F32, binding.F16, binding.BF16])
def test_kept_features_take_no_memory_of_their_own(L, H, hidden, E, interp, N, full, dtype):  # noqa: F811
    """What the forward of a 16-bit model keeps for the backward does not make
    the workspace larger: from 65,536 backward queries on, it grows by no more
    per point than the order, rank and radiance of every query and the seeds,
    nodes, coordinates, positions (paper's scheme) and dh of every backward
    query take side by side."""
    t, m = _tree(dtype=dtype), _mlp(K0=24 + E, H=H, n_layers=hidden + 1, dtype=dtype)
    t.interp = interp

    def size(B):
        b = binding._Batch()
        b.B, b.N, b.grad_through_rhs = B, N, full
        b.x = b.dir = b.Le = b.n = b.wo = b.albedo = b.rough = b.x2 = b.dir2 = b.wi = 0x5000
        if E:
            b.attr = b.attr2 = 0x5000
        n = C.c_size_t(0)
        assert L.oo_residual_workspace_bytes(C.byref(t), C.byref(m), C.byref(b), C.byref(n)) == 0, L.oo_last_error()
        return n.value

    backward = 1 + N if full else 1
    per_point = (1 + N) * (4 + 4 + 12) + backward * (12 + 3 * 4 * (8 if interp else 1) + 8 + 16 * interp + 4 * 24)
    per_point += 64 * 8 / 256  # loss partials: one of 8 bytes per 256 threads, at most 64 threads a point
    lo, hi = 1 << 17, 1 << 20
    assert size(hi) - size(lo) <= (hi - lo) * per_point + 16 * 256
