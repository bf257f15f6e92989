"""The dedup over the sizes at which its route changes (one block, tiles of 2048
and 4096 keys, the inverse index by buckets) and over ID ranges of one to four
radix passes: bit-exact against torch's unique and stable argsort.  Every route
also reports an ID outside its range, and its workspace holds what the size
function says for a larger batch."""
import pytest
import torch

from paper_1711_06505_amd import ams

pytestmark = pytest.mark.gpu


def buffers(n):
    new = lambda k: torch.full((k,), -7, dtype=torch.int32, device="cuda")  # noqa: E731
    return [new(max(n, 1)), new(max(n, 1)), new(max(n, 1)), new(n + 1), new(1), new(1)]


def draw(n, n_ids, law):
    g = torch.Generator(device="cuda").manual_seed(n + n_ids)
    if law == "one":
        return torch.full((n,), n_ids - 1, dtype=torch.int32, device="cuda")
    if law == "hot":            # half of the occurrences on three IDs
        ids = torch.randint(0, n_ids, (n,), generator=g, device="cuda", dtype=torch.int64)
        hot = torch.randint(0, min(3, n_ids), (n,), generator=g, device="cuda")
        return torch.where(torch.rand(n, generator=g, device="cuda") < 0.5, hot, ids).int()
    return torch.randint(0, n_ids, (n,), generator=g, device="cuda", dtype=torch.int64).int()


def check(n, n_ids, law, ws_n=None, noalloc=False):
    print(f"dedup n={n} n_ids={n_ids} {law}", flush=True)
    ids = draw(n, n_ids, law)
    o = buffers(n)
    if noalloc:
        ams.ams_dedup_noalloc(ids, n_ids, *o)
    else:
        ws = torch.full((ams.ams_dedup_workspace(ws_n or n, n_ids),), 255, dtype=torch.uint8, device="cuda")
        ams.ams_dedup(ids, n_ids, *o, ws)
    torch.cuda.synchronize()
    uniq, inv, count = torch.unique(ids, return_inverse=True, return_counts=True)
    n_u = uniq.numel()
    assert int(o[5]) == 0 and int(o[4]) == n_u
    assert torch.equal(o[0][:n_u], uniq)
    assert torch.equal(o[1], inv.int())
    assert torch.equal(o[2], torch.argsort(ids, stable=True).int())
    assert torch.equal(o[3][1:n_u + 1], torch.cumsum(count, 0).int()) and int(o[3][0]) == 0


@pytest.mark.parametrize("n", [1, 63, 64, 65, 1023, 1024, 1025, 2048, 2049, 4096, 4097, 8191, 8192, 8193, 16385])
@pytest.mark.parametrize("n_ids,law", [(1, "any"), (2, "any"), (200, "hot"), (70_000, "any"), (2_000_000, "hot"),
                                       (2**31 - 1, "any"), (5000, "one")])
def test_small_and_tiled(n, n_ids, law):
    check(n, n_ids, law)
    check(n, n_ids, law, noalloc=True)


@pytest.mark.parametrize("n", [2**20 - 1, 2**20, 2**20 + 4097, 2**21 - 1, 2**21, 2**21 + 32769, 2**24 + 1])
@pytest.mark.parametrize("n_ids,law", [(2, "any"), (300, "any"), (2_000_000, "hot"), (2**31 - 1, "any")])
def test_wide_and_buckets(n, n_ids, law):
    check(n, n_ids, law)


@pytest.mark.parametrize("n,ws_n", [(2**20 - 1, 2**20), (8193, 2**21), (100, 8192)])
def test_workspace_serves_smaller_batches(n, ws_n):
    for n_ids in (100, 1000, 70_000):
        check(n, n_ids, "hot", ws_n=ws_n)


@pytest.mark.parametrize("n", [70, 5000, 20_000, 2**20 + 5, 2**21 + 5])
@pytest.mark.parametrize("bad", [1000, -1, 2**31 - 1])
def test_out_of_range(n, bad):
    print(f"dedup range n={n} bad={bad}", flush=True)
    ids = draw(n, 1000, "any")
    ids[n // 2] = bad
    o = buffers(n)
    ws = torch.empty(ams.ams_dedup_workspace(n, 1000), dtype=torch.uint8, device="cuda")
    ams.ams_dedup(ids, 1000, *o, ws)
    torch.cuda.synchronize()
    assert ams.STATUS[int(o[5])] == "AMS_ERR_ID_RANGE"
    ids[n // 2] = 999
    ams.ams_dedup(ids, 1000, *o, ws)
    torch.cuda.synchronize()
    assert int(o[5]) == 0
