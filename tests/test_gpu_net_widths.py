"""GPU parity of the CTR model and the pre-rank towers at the widths where their
matrix-instruction layers can go wrong: layers of one unit, widths that are not
multiples of 4, of 16 or of 64, the widest layers, one sample and ragged last
blocks, towers of different depths, and the pair of towers whose backwards
have to take turns in LDS.  Against the float64 oracle at 1e-4, as the other
tests of these calls."""
import numpy as np
import pytest
import torch

from oracle import oracle
from paper_1711_06505_amd import ams
from tests.parity import assert_close
from tests.test_gpu_prerank import F32, check_net, cuda, dev_list, grads_like, net_params, run_dssm, split

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dims,B,widths,prelu", [
    ((1, 1, 2), 1, (1,), (True,)),
    ((3, 5, 2), 15, (1, 2), (False,)),
    ((17, 33, 7, 5), 16, (17,), (True, True)),
    ((63, 65, 15, 2), 31, (60, 3), (True, False)),
    ((64, 64, 64, 8), 33, (64,), (False, False)),
    ((66, 130, 17, 3), 100, (13, 53), (False, True)),
    ((127, 255, 254, 7), 47, (127,), (True, True)),
    ((128, 256, 256, 8), 1000, (16,) * 8, (True, True)),
])
def test_ctr_widths(dims, B, widths, prelu):
    print(f"ctr widths {dims} B={B}", flush=True)
    rng = np.random.default_rng(sum(dims) + B)
    Ws, bs, sl = net_params(rng, dims, prelu)
    X = (rng.standard_normal((B, dims[0])) * 0.8).astype(np.float32)
    labels = rng.integers(0, dims[-1], B).astype(np.int32)
    ref = oracle.ctr_act_fwd_bwd(X, labels, Ws, bs, sl)
    fields = split(X, widths)
    dfs = [torch.full_like(f, 7.0) for f in fields]
    dW, db, ds = grads_like(Ws, bs, sl)
    loss, prob = torch.zeros(1, device="cuda"), torch.zeros((B, dims[-1]), device="cuda")
    net = ams.make_ctr(dims)
    ws = torch.full((max(ams.ams_ctr_workspace(net, B), 256),), 255, dtype=torch.uint8, device="cuda")
    ams.ams_ctr_fwd_bwd(net, fields, cuda(labels), dev_list(Ws), dev_list(bs), loss, prob, dW, db, dfs, ws,
                        slopes=dev_list(sl), dslopes=ds)
    torch.cuda.synchronize()
    assert abs(loss.item() - ref["loss"]) <= F32 * max(1.0, abs(ref["loss"]))
    assert_close(prob, ref["prob"], F32, "prob")
    assert_close(torch.cat(dfs, 1), ref["dX"], F32, "dX")
    check_net("ctr", dW, db, ds, ref)


@pytest.mark.parametrize("user_dims,ad_dims,B", [
    ((1, 1), (1, 1), 3),
    ((17, 33, 5), (31, 5), 40),
    ((65, 127, 63, 64), (128, 64), 17),
    ((116, 213, 220, 4), (89, 194, 159, 4), 70),    # side by side they need more than 160 KB
])
def test_dssm_widths(user_dims, ad_dims, B):
    print(f"dssm widths {user_dims} {ad_dims} B={B}", flush=True)
    rng = np.random.default_rng(B)
    user = net_params(rng, user_dims, [True] * (len(user_dims) - 2))
    ad = net_params(rng, ad_dims, [True] * (len(ad_dims) - 2))
    Xu = (rng.standard_normal((B, user_dims[0])) * 0.8).astype(np.float32)
    Xa = (rng.standard_normal((B, ad_dims[0])) * 0.8).astype(np.float32)
    labels = (rng.random(B) < 0.3).astype(np.int32)
    ref = oracle.dssm_fwd_bwd(Xu, Xa, labels, user, ad)
    loss, prob, gu, ga, dXu, dXa = run_dssm(user_dims, ad_dims, (user_dims[0],), (ad_dims[0],), Xu, Xa, labels, user, ad)
    assert abs(loss.item() - ref["loss"]) <= F32 * max(1.0, abs(ref["loss"]))
    assert_close(prob, ref["prob"], F32, "prob")
    assert_close(dXu, ref["user"]["dX"], F32, "user dX")
    assert_close(dXa, ref["ad"]["dX"], F32, "ad dX")
    check_net("user", *gu, ref["user"])
    check_net("ad", *ga, ref["ad"])
