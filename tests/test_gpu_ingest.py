"""Ingestion of inputs on either side of what the memory-side cache holds: aligned rows whose pieces share few lines are read past the caches, four columns a thread."""
import pytest
import torch

import paper_2508_21230_amd as pkg

pytestmark = pytest.mark.gpu

CACHED = (256 << 20) // 4  # values


@pytest.mark.parametrize("n,d,ld,offset", [
    (CACHED // 100, 100, 100, 0),      # the last size that the caches are used for
    (CACHED // 100 + 1, 100, 100, 0),  # past the caches
    (CACHED // 100 + 1, 100, 100, 1),  # the same with rows that are not 16-byte aligned: four columns a thread, through the caches
    (CACHED // 101 + 2, 101, 101, 0),  # ... by their stride
    (CACHED // 70 + 3, 70, 76, 0),     # aligned, the last four columns of a row cut off, stride and padding wider than a row
    (CACHED // 192 + 1, 192, 192, 0),  # 48 chunks a row: sixteen threads side by side
    (CACHED // 32 + 1, 32, 32, 0),     # few coordinates: eight columns a thread
    (CACHED // 33 + 1, 33, 36, 0),
    (CACHED // 300 + 1, 300, 300, 0),  # pieces of rows that share lines: eight columns a thread, through the caches
    (CACHED // 324 + 1, 324, 324, 0),  # fewer of those: past them
    (CACHED // 324 * 15 // 8 + 9, 324, 324, 0),  # ... but not as large
    (CACHED // 192 + 1, 192, 192, 4),  # whole lines but for the first row's place
    (CACHED // 1000 + 1, 1000, 1000, 0),
])
def test_conversion_by_size_and_alignment(n, d, ld, offset):
    """Every step rounded in FP32, then to FP16: to the bit."""
    print(f"ingest n={n} d={d} ld={ld} offset={offset}", flush=True)
    gen = torch.Generator(device="cuda").manual_seed(n)
    flat = torch.randn(n * ld + offset, generator=gen, device="cuda")
    flat[::1001] *= 1e5  # some overflow FP16
    X = flat[offset:].view(n, ld)[:, :d]
    center = torch.randn(d, generator=gen, device="cuda")
    got = pkg.EJoin(0).convert_f32(X, scale=1.7, center=center)
    assert got.shape == (n, (d + 63) // 64 * 64) and not got[:, d:].any()
    for r in range(0, n, 1 << 18):
        want = ((X[r:r + (1 << 18)] - center) * 1.7).half()
        assert torch.equal(got[r:r + (1 << 18), :d].view(torch.int16), want.view(torch.int16))


# the last set normed from its first point on and the first normed from its last (240 MB of rows), ragged
@pytest.mark.parametrize("n,d", [(1966080, 20), (1966081, 20), (2200003, 64), (300001, 400)])
def test_norms_in_either_order_of_the_points(n, d):
    """Those of parts of the set, to the bit."""
    print(f"norms n={n} d={d}", flush=True)
    e = pkg.EJoin(0)
    gen = torch.Generator(device="cuda").manual_seed(n)
    X = e.convert_f32(torch.randn(n, d, generator=gen, device="cuda"))
    s = e.norms(X, d=d)
    for r in range(0, n, 99991):
        assert torch.equal(s[r:r + 99991], e.norms(X[r:r + 99991], d=d))
