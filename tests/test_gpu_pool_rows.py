"""The pooling backward against plain float64, with its rows packed and read where
they are (the rule between the two is checked on both sides): every row width
(columns short of, at and past the 12, 16 and 32 that a packed half holds),
chunks of the stable order that are full, short by one and over by one, samples
without behaviors, ads without an upstream gradient, a capacity below the unique
count, and the add into a given dE.

dE is a float32 sum of up to n products (1e-4 of the tensor's scale, as the other
parity tests)."""
import pytest
import torch

from paper_1711_06505_amd import ams
from tests.parity import assert_close

pytestmark = pytest.mark.gpu


def batch(B, n_occ, n_ids, g):
    n_beh = n_occ - B
    cut = torch.randint(0, n_beh + 1, (B - 1,), generator=g, device="cuda").sort().values
    seg = torch.cat([cut.new_zeros(1), cut, cut.new_full((1,), n_beh)])
    ids = (torch.rand(n_occ, generator=g, device="cuda") ** 3 * n_ids).long()
    uniq, inv = torch.unique(ids, return_inverse=True)
    perm = torch.sort(inv, stable=True).indices
    off = torch.cat([inv.new_zeros(1), torch.bincount(inv, minlength=uniq.numel()).cumsum(0)])
    sample = torch.repeat_interleave(torch.arange(B, device="cuda"), seg.diff())
    return n_beh, seg, inv, perm, off, sample, uniq.numel()


@pytest.mark.parametrize("mode", ["sum", "max", "att", "query"])
@pytest.mark.parametrize("B,n_occ,D", [
    (1, 1, 12), (3, 63, 1), (5, 64, 12), (7, 65, 12), (9, 257, 11), (40, 1000, 4), (64, 3001, 13), (33, 2048, 16),
    (50, 2047, 17), (21, 1025, 31), (70, 5000, 32), (300, 70_000, 12),
])
def test_pool_backward_rows(mode, B, n_occ, D):
    check(mode, B, n_occ, D)


# Where the rule between packed rows and rows read where they are changes its
# answer: mode, D, samples, and the fewest behaviors that are packed (with one
# behavior less they are not).  Mean lists of 10, 20, 25, 40 and 100, batches of
# 150,000 to 2^21, rows in whole 16-byte pieces and not.
@pytest.mark.parametrize("mode,D,B,n_beh", [
    ("sum", 8, 9000, 2**20), ("sum", 3, 10_487, 1_048_700), ("sum", 10, 7001, 150_000), ("sum", 11, 52_431, 524_310),
    ("sum", 13, 2501, 20_008), ("sum", 12, 20_001, 2**20), ("sum", 16, 9999, 2**19), ("sum", 20, 2**10, 2**20),
    ("sum", 32, 52_429, 524_290), ("max", 5, 20_973, 524_325), ("max", 8, 1000, 2**19), ("max", 12, 15_007, 150_070),
    ("max", 17, 2501, 20_008), ("max", 20, 2000, 150_000), ("max", 32, 2000, 20_000), ("att", 4, 8001, 2**20),
    ("att", 6, 3333, 150_000), ("att", 12, 15_003, 150_030), ("att", 16, 2049, 150_000), ("att", 24, 16_384, 163_840),
    ("att", 28, 5001, 150_000), ("att", 20, 4097, 2**21), ("query", 12, 9001, 150_000),
    ("query", 20, 52_429, 2_097_160), ("query", 32, 1025, 150_000),
])
def test_pool_backward_routes(mode, D, B, n_beh):
    for n, kernel in ((n_beh, "pool_bwd_seg"), (n_beh - 1, "pool_bwd_seg_rows")):
        ams.ams_timing_read()
        ams.ams_timing_enable(True)
        try:
            check(mode, B, n + B, D, full_only=True)
            ran = ams.ams_timing_read()
        finally:
            ams.ams_timing_enable(False)
        assert kernel in ran and len({"pool_bwd_seg", "pool_bwd_seg_rows"} & set(ran)) == 1


def check(mode, B, n_occ, D, full_only=False):
    print(f"pool rows {mode} B={B} n_occ={n_occ} D={D}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(n_occ + D)
    n_beh, seg, inv, perm, off, sample, n_u = batch(B, n_occ, max(2, n_occ // 3), g)
    rand = lambda *s: torch.randn(s, generator=g, device="cuda")  # noqa: E731
    E, U, A, dU, dA, dE0 = rand(n_u, D), rand(B, D), rand(B, D), rand(B, D), rand(B, D), rand(n_u, D)
    if n_occ % 2 == 0 or mode == "query":
        dA = None
    w = torch.rand(max(n_beh, 1), generator=g, device="cuda")
    arg = seg[:-1, None] + (torch.rand((B, D), generator=g, device="cuda") * seg.diff()[:, None]).long()
    arg = torch.where(seg.diff()[:, None] > 0, arg, -1).int()
    # float64: each occurrence's gradient, then the sums
    d, e = dU.double()[sample], E.double()[inv[:n_beh]]
    ad = torch.zeros((B, D), dtype=torch.float64, device="cuda") if dA is None else dA.double()
    dq = None
    if mode == "sum":
        v = d
    elif mode == "max":
        v = torch.where(arg[sample] == torch.arange(n_beh, device="cuda")[:, None], d, 0.0)
    else:
        ds = w[:n_beh].double() * ((d * e).sum(1) - (dU.double() * U.double()).sum(1)[sample])
        v = w[:n_beh].double()[:, None] * d + ds[:, None] * A.double()[sample]
        dq = torch.zeros((B, D), dtype=torch.float64, device="cuda").index_add_(0, sample, ds[:, None] * e)
        if mode == "att":
            ad = ad + dq
    want = torch.zeros((n_u, D), dtype=torch.float64, device="cuda").index_add_(0, inv, torch.cat([v, ad]))

    i32 = lambda t: t.int().contiguous()  # noqa: E731
    nu = torch.tensor([n_u], dtype=torch.int32, device="cuda")
    for cap in {n_u} if full_only else {n_u, max(1, n_u // 2), n_u + 9}:
        rows = min(cap, n_u)
        Ec = torch.zeros((cap, D), device="cuda")
        Ec[:rows] = E[:rows]
        dE = torch.full((cap, D), float("nan"), device="cuda")
        ws = torch.full((ams.ams_pool_workspace("att" if mode == "query" else mode, B, n_beh, D, cap),), 255,
                        dtype=torch.uint8, device="cuda")
        ix = i32(seg), n_beh, i32(inv), i32(perm), i32(off), nu, cap, Ec
        if mode == "query":
            dQ = torch.full((B, D), float("nan"), device="cuda")
            dE[:rows] = dE0[:rows]
            ams.ams_pool_query_bwd(*ix, A, U, w, dU, dQ, dE, True, ws)
        else:
            ams.ams_pool_bwd(mode, *ix, U, A, {"sum": None, "max": arg, "att": w}[mode], dU, dA, dE, ws)
        torch.cuda.synchronize()
        ref = want + (dE0.double() if mode == "query" else 0.0)
        if cap < n_u and mode in ("att", "query"):
            # (dropped occurrences read a zero row: their own score gradients differ, and so the ads')
            keep = torch.ones(n_u, dtype=torch.bool, device="cuda")
            if mode == "att":
                keep[inv[n_beh:]] = False
            keep = keep[:rows]
            assert_close(dE[:rows][keep], ref[:rows][keep], 1e-4, f"dE cap={cap}")
            continue
        assert_close(dE[:rows], ref[:rows], 1e-4, f"dE cap={cap}")
        if mode == "query":
            assert_close(dQ, dq, 1e-4, "dQ")
