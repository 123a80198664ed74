"""GPU parity at the sizes where a kernel's tiling or a dispatch rule has its edges: tiles plus or minus one,
remainders, the smallest layers, both sides of a line between two variants."""
import numpy as np
import pytest

import workloads
from test_gpu_parity import both_configs, dev, rel_l2, xb  # noqa: F401 (fixture)

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


# M, K, N: odd weight counts (no 16-byte rows), one batch partial, the 8- and 32-group reductions, many weights
@pytest.mark.parametrize("M,K,N", [(5, 3, 7), (9000, 9, 5), (40000, 16, 12), (3000, 33, 65), (33, 1023, 513)])
@pytest.mark.parametrize("pair", [False, True])
def test_update_write(xo, xb, M, K, N, pair):
    W, X, dY = workloads.layer_tensors_np(workloads.Gemm("t", K, N, M, False, 1), seed=M + K)
    co, cg = both_configs(xo, xb, flags=xo.UPD_NL | xo.UPD_NOISE, upd_nl_v=0.3, upd_noise_gamma=2.0, seed=5)
    w_max = 2.0 * float(np.abs(W).max())
    Wg = dev(W.copy())
    if pair:
        Gp, Gn = xo.pair_init(W, w_max)
        Gpg, Gng = dev(Gp.copy()), dev(Gn.copy())
        want = xo.update_pair(co, Gp, Gn, X, dY, w_max, 1.0 / w_max, 0.01, step=4)[2]
        xb.update_pair(cg, Gpg, Gng, Wg, dev(X), dev(dY), w_max, 1.0 / w_max, 0.01, step=4)
    else:
        want = xo.update(co, W, X, dY, w_max, 1.0 / w_max, 0.01, step=4)
        xb.update(cg, Wg, dev(X), dev(dY), w_max, 1.0 / w_max, 0.01, step=4)
    torch.cuda.synchronize()
    assert rel_l2(Wg.cpu().numpy() - W, want - W) <= 1e-3

