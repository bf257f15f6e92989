"""The split-float32 mode's first weight gradient over float32's whole range: the
backward of the same saved layers in both float32 modes.  Gradients and feature
rows down to float32's smallest normals keep float32's precision, and where a
value or a sum leaves the range (infinities, NaN, values that would round to
infinity in bf16) the same elements are infinite or NaN as in the float32 mode."""
import pytest
import torch

from paper_1711_06505_amd import ams
from tests.test_gpu_shares import model

pytestmark = pytest.mark.gpu
DIMS = (512, 256, 64, 12)


def dw1(dtype, T, W, uniq, H1, H2, E, dE):
    n = uniq.numel()
    mlp = ams.make_mlp(DIMS, dtype)
    n_uniq = torch.full((1,), n, dtype=torch.int32, device="cuda")
    dW, db = [torch.full_like(w, 7.0) for w in W], [torch.full((w.shape[0],), 7.0, device="cuda") for w in W]
    ws = torch.full((ams.ams_embed_workspace(mlp, n),), 255, dtype=torch.uint8, device="cuda")
    ams.ams_embed_bwd(mlp, T, uniq, n_uniq, n, W, H1, H2, E, dE, dW, db, ws)
    torch.cuda.synchronize()
    return dW[0]


def layers(n):
    """Saved hidden layers with about half of the units active."""
    T, W, _, uniq, dE = model(DIMS, "f32", n)
    g = torch.Generator(device="cuda").manual_seed(n)
    H1, H2 = [torch.randn((n, d), generator=g, device="cuda").clamp_min_(0) for d in DIMS[1:3]]
    return T, W, uniq, H1, H2, torch.zeros((n, DIMS[-1]), device="cuda"), dE


def exact(T, W, uniq, H1, H2, dE):
    d2 = (dE.double() @ W[2].double()) * (H2 > 0)
    return ((d2 @ W[1].double()) * (H1 > 0)).t() @ T[uniq.long()].double()


# scale of dE, scale of the features (powers of two: the float32 products are the same but for them)
@pytest.mark.parametrize("s_e,s_t", [(0, 0), (-90, 0), (-100, 0), (-110, 0), (-115, 0), (-120, 0), (0, -100), (0, -115),
                                     (60, -122), (-60, -60), (90, 0), (100, 0), (110, 0), (40, 60), (0, 120)])
@pytest.mark.parametrize("n", [1, 333])
def test_precision_over_the_range(n, s_e, s_t):
    print(f"split dW1 range n={n} dE 2^{s_e} T 2^{s_t}", flush=True)
    T, W, uniq, H1, H2, E, dE = layers(n)
    T, dE = T * 2.0 ** s_t, dE * 2.0 ** s_e
    ref = exact(T, W, uniq, H1, H2, dE)
    err = {}
    for dtype in ("f32", "f32x3"):
        got = dw1(dtype, T, W, uniq, H1, H2, E, dE)
        assert torch.isfinite(got).all()
        err[dtype] = float((got.double() - ref).norm() / ref.norm())
    assert err["f32x3"] <= max(1.05 * err["f32"], 1.5e-7), err     # (2^-23: a sum of a few products)


def one_unit(W):
    """Weights through which dE[u][0] reaches unit 0 alone, as it is."""
    for w in W[1:]:
        w.zero_()
        w[0, 0] = 1.0


@pytest.mark.parametrize("what", ["inf", "-inf", "nan", "3.4e38", "3.39e38", "5.2e33", "T inf", "T nan", "T 3.4e38",
                                  "T -3.4e38 dE 0.5", "sum"])
@pytest.mark.parametrize("n,u", [(40, 7), (333, 332)])
def test_out_of_range_as_float32(n, u, what):
    print(f"split dW1 out of range n={n} u={u} {what}", flush=True)
    T, W, uniq, H1, H2, E, dE = layers(n)
    H1[u], H2[u] = 1.0, 1.0
    one_unit(W)
    if what == "sum":                                      # finite products whose sum is not
        dE[u, 0], T[uniq[u].long(), 100] = 3e38, 0.9
        dE[3, 0], T[uniq[3].long(), 100] = 3e38, 0.9
        H1[3], H2[3] = 1.0, 1.0
    elif what.startswith("T"):
        w = what.split()
        T[uniq[u].long(), 100] = float(w[1])
        if len(w) > 2:
            dE[u, 0] = float(w[3])
    else:
        dE[u, 0] = float(what)
    got = {d: dw1(d, T, W, uniq, H1, H2, E, dE) for d in ("f32", "f32x3")}
    f, x = got["f32"], got["f32x3"]
    assert torch.equal(torch.isnan(f), torch.isnan(x))
    assert torch.equal(torch.isinf(f), torch.isinf(x)) and torch.equal(f[torch.isinf(f)], x[torch.isinf(x)])
    ok = torch.isfinite(f)
    assert float((f - x)[ok].double().norm()) <= 1e-5 * float(f[ok].double().norm())
