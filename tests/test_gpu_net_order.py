"""The order of the CTR model's forward sums, which decides the side that a
hidden unit within rounding of zero takes: the bias is set so that every unit's
sum is zero or a rounding error of its terms, and the units that let a gradient
through have to be those that the stated order (a part's terms in the order of
k, each product and sum rounded once; the parts in order onto the bias) leaves
above zero.  The oracle is that order in 80-bit floats, rounded to 32 bits after
each term: exact products (48 bits), so no tolerance is needed."""
import numpy as np
import pytest
import torch

from paper_1711_06505_amd import ams
from tests.test_gpu_prerank import cuda, dev_list, grads_like, net_params

pytestmark = pytest.mark.gpu


def parts(x, W):
    """The rounded sum of each part, [parts][O]."""
    O, K = W.shape
    p = max(1, min(512 // O, (K + 15) // 16))
    width = ((K + p - 1) // p + 3) & ~3
    out = []
    for k0 in range(0, K, width):
        acc = np.zeros(O, np.float32)
        for k in range(k0, min(K, k0 + width)):
            acc = (np.longdouble(x[k]) * W[:, k].astype(np.longdouble) + acc).astype(np.float32)
        out.append(acc)
    return out


@pytest.mark.parametrize("K,O", [(16, 256), (3, 256), (72, 200), (70, 131), (128, 80), (127, 256), (65, 17), (128, 1)])
def test_ctr_forward_order(K, O):
    print(f"ctr order {K} {O}", flush=True)
    rng = np.random.default_rng(K + O)
    dims = (K, O, 2)
    Ws, bs, sl = net_params(rng, dims, (False,))
    x = rng.standard_normal((1, K)).astype(np.float32)
    sums = parts(x[0], Ws[0])
    bs[0] = -np.sum(np.stack(sums).astype(np.longdouble), axis=0).astype(np.float32)
    z = bs[0].copy()
    for s in sums:
        z = z + s
    dW, db, ds = grads_like(Ws, bs, sl)
    loss, prob = torch.zeros(1, device="cuda"), torch.zeros((1, 2), device="cuda")
    net = ams.make_ctr(dims)
    ws = torch.full((max(ams.ams_ctr_workspace(net, 1), 256),), 255, dtype=torch.uint8, device="cuda")
    ams.ams_ctr_fwd_bwd(net, [cuda(x)], cuda(np.zeros(1, np.int32)), dev_list(Ws), dev_list(bs), loss, prob, dW, db,
                        [torch.empty((1, K), device="cuda")], ws, slopes=dev_list(sl), dslopes=ds)
    torch.cuda.synchronize()
    np.testing.assert_array_equal(db[0].cpu().numpy() != 0, z > 0)
