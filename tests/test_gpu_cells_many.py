"""Cells in groups of several tensors beyond the line for single ones: the same blobs as in a group that has none (one of whose
tensors is too large for them), by tensor count, code width and ragged size.  test_gpu_cells.py compares cells with the oracle."""
import pytest
import torch

import paper_2406_11257_amd as X

pytestmark = pytest.mark.gpu
BEYOND = 28_000_003                                         # a bucket of a third of it does not fit a workgroup's registers


def tensor(n, seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    Wp = torch.randn(n, device="cuda", generator=g) * 0.02
    u = torch.rand(n, device="cuda", generator=g) - 0.5
    W = Wp - torch.sign(u) * torch.log1p(-2 * u.abs().clamp_(max=0.49999997)) * 1e-4
    m = torch.randn(n, device="cuda", generator=g) * 5e-5
    v = m * m * torch.exp(torch.randn(n, device="cuda", generator=g)) + 1e-16
    return Wp, W, m, v


def compress(ctx, tensors, nbits):
    items = [(*t, torch.zeros(X.excp_blob_bound(t[0].numel(), nbits), dtype=torch.uint8, device="cuda"), torch.zeros_like(t[0])) for t in tensors]
    ctx.excp_compress_tensors(items, 5e-5, 2.0, nbits, 10)
    return items, ctx.excp_collect()[1]


@pytest.mark.parametrize("sizes, nbits", [([13_500_001, 14_600_003], 4), ([9_000_001, 8_500_077, 11_000_000, 9_999_999], 3), ([6_000_005] * 5, 6),
                                          ([3_000_001 + 64 * i for i in range(12)], 8), ([131_071, 131_073, 20_000_001, 25 << 20], 7)])
def test_blobs_are_those_of_a_group_without_cells(sizes, nbits):
    tensors = [tensor(n, i) for i, n in enumerate(sizes)]
    ctx = X.Context(BEYOND, sum(sizes) + BEYOND)
    with_cells, a = compress(ctx, tensors, nbits)
    without, b = compress(ctx, tensors + [tensor(BEYOND, 99)], nbits)
    ctx.close()
    for x, y, p, q in zip(with_cells, without, a, b):
        assert (p.status, p.blob_bytes, p.n_w, p.n_o) == (0, q.blob_bytes, q.n_w, q.n_o)
        assert torch.equal(x[4], y[4]) and torch.equal(x[5].view(torch.int32), y[5].view(torch.int32))
