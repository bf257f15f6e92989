"""GPU parity of the embedding model, forward and backward, over the numbers of
unique images at which the stream-K first layer's plan changes: one row to
several tiles, tiles cut into many shares, shares that follow the tile
boundaries and shares that cross them, workers left idle, one whole tile per
worker.  Reference: the same model in plain PyTorch float64.

Float32 and split-float32 results are float32 sums of at most 4096 products
(1e-4 of the tensor's scale, as the other parity tests); bf16 storage takes the
stored values as exact, so E meets the same bound and the weight gradients,
whose operands are rounded to bf16, 2e-2."""
import pytest
import torch

from paper_1711_06505_amd import ams
from tests.parity import RTOL, assert_close

pytestmark = pytest.mark.gpu


def model(dims, dtype, n, seed=5):
    g = torch.Generator(device="cuda").manual_seed(seed)
    store = torch.bfloat16 if dtype == "bf16" else torch.float32
    T = torch.empty((n + 7, dims[0]), device="cuda").normal_(generator=g).clamp_min_(0).to(store)
    W = [(torch.randn((o, i), generator=g, device="cuda") * (2.0 / (i + o)) ** 0.5).to(store)
         for i, o in zip(dims[:-1], dims[1:])]
    b = [torch.rand(o, generator=g, device="cuda") * 0.2 - 0.1 for o in dims[1:]]
    uniq = torch.randperm(n + 7, generator=g, device="cuda")[:n].sort().values.int()
    dE = torch.randn((n, dims[-1]), generator=g, device="cuda")
    return T, W, b, uniq, dE


def run(dims, dtype, T, W, b, uniq, dE, cap):
    n = uniq.numel()
    mlp = ams.make_mlp(dims, dtype)
    new = lambda *s, **k: torch.full(s, float("nan"), device="cuda", **k)  # noqa: E731
    n_uniq = torch.full((1,), n, dtype=torch.int32, device="cuda")
    ids = torch.full((cap,), -1, dtype=torch.int32, device="cuda")
    ids[:n] = uniq
    H1 = new(cap, dims[1], dtype=torch.bfloat16 if dtype == "bf16" else torch.float32)
    H2 = new(cap, dims[2]) if len(dims) == 4 else None
    E, up = new(cap, dims[-1]), new(cap, dims[-1])
    up[:n] = dE
    dW, db = [new(*w.shape) for w in W], [new(*x.shape) for x in b]
    ws = torch.empty(ams.ams_embed_workspace(mlp, cap), dtype=torch.uint8, device="cuda")
    ams.ams_embed_fwd(mlp, T, ids, n_uniq, cap, W, b, H1, H2, E, ws)
    ams.ams_embed_bwd(mlp, T, ids, n_uniq, cap, W, H1, H2, E, up, dW, db, ws)
    torch.cuda.synchronize()
    return H1[:n], H2[:n] if H2 is not None else None, E[:n], dW, db


def reference(T, W, b, uniq, dE, H1, H2):
    """Plain float64.  The backward takes the masks of the given hidden layers
    (a unit within rounding of zero may be taken either way)."""
    x = T[uniq.long()].double()
    Wd = [w.double() for w in W]
    h = [x]
    for l, (w, c) in enumerate(zip(Wd, b)):
        z = h[-1] @ w.t() + c.double()
        h.append(z.clamp_min(0) if l + 1 < len(W) else z)
    masks = [H1 > 0] + ([H2 > 0] if H2 is not None else [])
    d, dW, db = dE.double(), [None] * len(W), [None] * len(W)
    for l in range(len(W) - 1, -1, -1):
        dW[l], db[l] = d.t() @ h[l], d.sum(0)
        if l:
            d = (d @ Wd[l]) * masks[l - 1]
    return h, dW, db


PAPER, SMALL = (4096, 256, 64, 12), (256, 256, 9)


@pytest.mark.parametrize("dtype", ["f32", "f32x3", "bf16"])
@pytest.mark.parametrize("dims,n,cap", [
    (PAPER, 1, 1), (PAPER, 33, 100), (PAPER, 128, 128), (PAPER, 129, 140),
    (PAPER, 1031, 1100),        # every tile in the most shares it may have
    (PAPER, 2049, 2049),        # 17 tiles: shares of 7 (bf16) and 4-row groups
    (PAPER, 6001, 6001),        # 47 tiles: float32 shares cross tile boundaries
    (PAPER, 12900, 12900),      # 101 tiles: two shares each in bf16 (202 workers)
    (PAPER, 18001, 18001),      # 141 tiles: shares cross tile boundaries in every type
    (PAPER, 30000, 30000),      # 235 tiles: one whole tile per worker in bf16
    (PAPER, 8192, 8192), (PAPER, 8193, 8193),   # tail backward: 256 blocks of 32 rows, 129 of 64
    (SMALL, 1, 5), (SMALL, 257, 300), (SMALL, 4000, 4000), (SMALL, 8193, 8200),
])
def test_embed_over_share_plans(dims, n, cap, dtype):
    print(f"shares {dims} n={n} cap={cap} {dtype}", flush=True)
    T, W, b, uniq, dE = model(dims, dtype, n)
    H1, H2, E, dW, db = run(dims, dtype, T, W, b, uniq, dE, cap)
    h, rW, rb = reference(T, W, b, uniq, dE, H1, H2)
    assert_close(H1, h[1], 1e-2 if dtype == "bf16" else 1e-4, "H1")
    assert_close(E, h[-1], 1e-4, "E", rows=True)
    for l in range(len(W)):
        assert_close(dW[l], rW[l], RTOL[dtype], f"dW{l + 1}")
        assert_close(db[l], rb[l], RTOL[dtype], f"db{l + 1}")


@pytest.mark.parametrize("dims,n,prelu", [
    ((4096, 256, 64, 12), 517, True), ((4096, 256, 64, 12), 3000, True), ((4096, 256, 33, 20), 700, False),
    ((256, 256, 32), 65, True), ((128, 256, 7), 1, False), ((4096, 256, 40, 17), 1300, True),
])
def test_split_weight_gradient(dims, n, prelu):
    """The split-float32 backward (dZ1 as three bf16 planes) with every form of
    the tail: two and three layers, narrow and wide outputs, PReLU; rows past the
    capacity's end, and IDs outside the table, which read as zero rows.  dW1's
    error stays within the float32 mode's."""
    print(f"split dW1 {dims} n={n} prelu={prelu}", flush=True)
    T, W, b, uniq, dE = model(dims, "f32", n)
    uniq[n // 2] = T.shape[0] + 5
    cap = n + 40
    g = torch.Generator(device="cuda").manual_seed(n)
    slopes = [torch.rand(d, generator=g, device="cuda") * 0.6 - 0.2 for d in dims[1:-1]] if prelu else None
    x = T[uniq.long().clamp_max(T.shape[0] - 1)].double()
    x[n // 2] = 0
    err = {}
    for dtype in ("f32", "f32x3"):
        mlp = ams.make_mlp(dims, dtype)
        new = lambda *s: torch.full(s, float("nan"), device="cuda")  # noqa: E731
        n_uniq = torch.full((1,), n, dtype=torch.int32, device="cuda")
        ids, up = torch.full((cap,), -1, dtype=torch.int32, device="cuda"), new(cap, dims[-1])
        ids[:n], up[:n] = uniq, dE
        H1, E = new(cap, dims[1]), new(cap, dims[-1])
        H2 = new(cap, dims[2]) if len(dims) == 4 else None
        dW, db = [new(*w.shape) for w in W], [new(*c.shape) for c in b]
        ds = [new(*a.shape) for a in slopes] if prelu else None
        ws = torch.full((ams.ams_embed_workspace(mlp, cap),), 255, dtype=torch.uint8, device="cuda")
        ams.ams_embed_fwd(mlp, T, ids, n_uniq, cap, W, b, H1, H2, E, ws, slopes=slopes)
        ams.ams_embed_bwd(mlp, T, ids, n_uniq, cap, W, H1, H2, E, up, dW, db, ws, slopes=slopes, dslopes=ds)
        torch.cuda.synchronize()
        # float64, on the saved hidden layers (pre-activations with PReLU) as the call's own inputs
        hid = [h[:n].double() for h in (H1, H2) if h is not None]
        d, rW, rs = dE.double(), [None] * len(W), [None] * (len(W) - 1)
        for l in range(len(W) - 1, -1, -1):
            if l < len(W) - 1:
                z = hid[l]
                if prelu:
                    rs[l] = (d * z.clamp_max(0)).sum(0)
                d = d * torch.where(z > 0, 1.0, slopes[l].double() if prelu else 0.0)
            h = x if l == 0 else hid[l - 1] if not prelu else torch.where(
                hid[l - 1] > 0, hid[l - 1], hid[l - 1] * slopes[l - 1].double())
            rW[l] = d.t() @ h
            if l:
                d = d @ W[l].double()
        for l in range(len(W)):
            assert_close(dW[l], rW[l], RTOL[dtype], f"{dtype} dW{l + 1}")
        for l in range(len(W) - 1):
            if prelu:
                assert_close(ds[l], rs[l], RTOL[dtype], f"{dtype} dslope{l + 1}")
        err[dtype] = float((dW[0].double() - rW[0]).norm() / rW[0].norm().clamp_min(1e-30))
    assert err["f32x3"] <= max(err["f32"], 1.5e-7), err     # (2^-23: a sum of a few products)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("cap", [300, 131072])      # tails after the stream-K and the row-split layer
@pytest.mark.parametrize("M,D", [(64, 12), (64, 10), (63, 32), (17, 4), (33, 1), (16, 29)])
def test_tail_output_widths(M, D, cap, dtype):
    """The last layer's widths and a middle layer that is no multiple of its
    blocks of 16, with E's rows on 16-byte boundaries and 4 bytes past them."""
    dims, n = (4096, 256, M, D), 261
    print(f"tail widths {dims} cap={cap} {dtype}", flush=True)
    T, W, b, uniq, dE = model(dims, dtype, n)
    mlp = ams.make_mlp(dims, dtype)
    n_uniq = torch.full((1,), n, dtype=torch.int32, device="cuda")
    ids = torch.full((cap,), -1, dtype=torch.int32, device="cuda")
    ids[:n] = uniq
    H1 = torch.empty((cap, 256), dtype=torch.bfloat16 if dtype == "bf16" else torch.float32, device="cuda")
    H2 = torch.empty((cap, M), device="cuda")
    ws = torch.empty(ams.ams_embed_workspace(mlp, cap), dtype=torch.uint8, device="cuda")
    h, _, _ = reference(T, W, b, uniq, dE, torch.zeros((n, 256), device="cuda"), torch.zeros((n, M), device="cuda"))
    for shift in (0, 1):
        buf = torch.full((cap * D + 1,), float("nan"), device="cuda")
        E = buf[shift:shift + cap * D].view(cap, D)
        ams.ams_embed_fwd(mlp, T, ids, n_uniq, cap, W, b, H1, H2, E, ws)
        torch.cuda.synchronize()
        assert_close(H2[:n], h[2], 1e-4, "H2")
        assert_close(E[:n], h[3], 1e-4, f"E shift={shift}", rows=True)
        assert bool(buf[shift + n * D:].isnan().all())
