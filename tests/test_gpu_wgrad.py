"""Weight gradients of the corrector at grids that do not fill the kernels'
4 x 4 x 32-cell tiles (and one that wraps its halo onto itself), against the
oracle fed the same BF16-rounded operands.

Tolerance: the products are exact in FP32 and at most 40^3 of them are summed,
so the sums differ by less than 1e-5; a hidden data gradient whose BF16
rounding falls the other way differs by 2^-9 in less than one element of a
thousand.  1e-3 holds both.
"""
import numpy as np
import pytest

from test_gpu_corrector import oracle_backward, oracle_forward, random_params, rel_l2, split_params, to_cf

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [4, 5, 31, 33, 40])
def test_gradients_on_partial_tiles_match_oracle(wdm, orc, n):
    rng = np.random.default_rng(n)
    net = wdm.Net(n)
    params = random_params(wdm, rng)
    wdm.wdm_net_set_params(net.handle, params)
    x = rng.standard_normal((n ** 3, 3)).astype(np.float32)
    dy = rng.standard_normal((n ** 3, 2)).astype(np.float32)
    wdm.wdm_net_forward(net.handle, torch.from_numpy(x).cuda())
    wdm.wdm_net_backward(net.handle, torch.from_numpy(dy).cuda())
    got = split_params(wdm.wdm_net_get_grads(net.handle))
    _, acts = oracle_forward(orc, params, x, n)
    ref = oracle_backward(orc, params, acts, to_cf(dy, n))
    for l in range(3):
        assert rel_l2(got[l][0], ref[l][0]) < 1e-3, l
        assert rel_l2(got[l][1], ref[l][1]) < 1e-3, l
    net.close()
