"""Cells inside the buckets (k_km_cells) and the iterations that use them, against the oracle, blob for blob: at the sizes
where a tensor or a bucket begins to have cells and where it no longer fits a workgroup, for each number of lanes and
centres, for buckets of one sign, of both, of more binary orders than the packed sums or any sums hold, for streams that
crowd one bucket beside others that do not, and in groups that go with and without cells."""
import numpy as np
import pytest

import oracle as O
import paper_2406_11257_amd as X
from gpu_util import gpu_compress

pytestmark = pytest.mark.gpu
f32 = np.float32


def draw(n, seed, kind):
    g = np.random.default_rng(seed)
    if kind == "one sign":
        d = g.gamma(0.5, 1e-4, n) + 1e-7
    elif kind == "both signs":
        d = g.normal(0, 1e-4, n)
    elif kind == "orders":                  # the middle bucket spans fifteen binary orders, others one
        d = g.normal(0, 1, n) * 2.0 ** -g.gamma(1.0, 3.0, n) * 1e-3
    elif kind == "far apart":               # most buckets span more than the sums hold
        d = 2.0 ** g.uniform(-120, -5, n) * g.choice([-1.0, 1.0], n)
    else:                                   # "crowded": nearly all in one bucket
        d = np.where(g.random(n) < 0.02, g.uniform(-1, 1, n) * 1e-4, 1e-4 * (1 + 1e-5 * g.standard_normal(n)))
    m = g.standard_normal(n) * 5e-5
    v = m * m * np.exp(g.standard_normal(n)) + 1e-16
    return np.zeros(n, f32), d.astype(f32), m.astype(f32), v.astype(f32)


def check(cases, nbits, iters, alpha=0.0, beta=0.0, flags=0):
    sizes = [c[0].size for c in cases]
    ctx = X.Context(max(sizes), sum(sizes))
    rc, out = gpu_compress(ctx, cases, alpha, beta, nbits, iters, flags=flags)
    assert rc == 0
    for c, o in zip(cases, out):
        assert o["blob"] == O.compress_step(*c, alpha, beta, nbits, iters, flags=flags).blob
    ctx.close()


@pytest.mark.parametrize("kind", ["one sign", "both signs", "orders", "far apart", "crowded"])
@pytest.mark.parametrize("nbits", [2, 4, 5, 8])
def test_tensors_with_cells(kind, nbits):
    for n in (131_071, 131_072, 262_145):
        print(kind, nbits, n, flush=True)
        check([draw(n, n + nbits, kind)], nbits, 3)


@pytest.mark.parametrize("n", [2_097_152, 2_097_153])
def test_buckets_on_both_sides_of_the_small_workgroup(n):
    check([draw(n, 3, "both signs"), draw(1000, 4, "one sign")], 4, 2)


def test_a_tensor_whose_buckets_take_more_samples():
    check([draw(14_800_001, 9, "both signs")], 4, 1, alpha=5e-5, beta=2.0)


def test_small_tensors_beside_large_ones():
    check([draw(n, n, k) for n, k in ((300_000, "both signs"), (5, "one sign"), (131_072, "crowded"), (4096, "orders"), (70_001, "far apart"))], 6, 3)


def test_more_elements_than_go_with_cells():
    # 26.3 M elements in all: the small one is compared, the others are there for the sum
    sizes = [9_000_000, 9_000_000, 8_000_000, 300_000]
    cases = [draw(n, i, "both signs") for i, n in enumerate(sizes)]
    ctx = X.Context(max(sizes), sum(sizes))
    rc, out = gpu_compress(ctx, cases, 5e-5, 2.0, 4, 2, want_recon=False)
    assert rc == 0 and out[3]["blob"] == O.compress_step(*cases[3], 5e-5, 2.0, 4, 2).blob
    ctx.close()


@pytest.mark.parametrize("sizes", [[2_097_152, 300_000], [4_000_000] * 3 + [300_000]], ids=["buckets", "survivors"])
def test_groups_that_turn_out_to_keep_too_much_for_cells(sizes):
    # (alpha is not 0, so that only the counts say that nearly everything is kept)
    cases = [draw(n, i, "both signs") for i, n in enumerate(sizes)]
    ctx = X.Context(max(sizes), sum(sizes))
    rc, out = gpu_compress(ctx, cases, 1e-9, 0.0, 4, 2, want_recon=False)
    assert rc == 0 and out[0]["stats"].n_o > 0.999 * sizes[0]
    for i in {len(sizes) - 1, 0 if sizes[0] < 3_000_000 else len(sizes) - 1}:
        assert out[i]["blob"] == O.compress_step(*cases[i], 1e-9, 0.0, 4, 2).blob
    ctx.close()


@pytest.mark.parametrize("n, seed", [(131_072, 2), (131_072, 5), (500_000, 1)])
def test_a_bucket_over_many_orders_with_a_large_cell_and_without(n, seed):
    # everything kept: the middle bucket of the residuals spans ten binary orders and its largest cell has some 230 of 513 values,
    # or sixteen orders and a cell of some 1000 of 1953
    check([draw(n, seed, "both signs")], 8, 3)


def with_zeros(n, zeros, sign):
    """Second moments of one sign, `zeros` of them zero (of the same sign): fewer than a bucket's share, so that they lie in the
    lowest (highest) bucket beside other values.  The ablations keep such elements."""
    Wp, W, m, v = draw(n, n + zeros, "both signs")
    v[np.random.default_rng(zeros).choice(n, zeros, replace=False)] = 0.0
    return Wp, W, m, (v if sign > 0 else -v)


@pytest.mark.parametrize("flags", [X.EXCP_FLAG_NO_W2M, X.EXCP_FLAG_NO_M2W])
@pytest.mark.parametrize("sign", [1, -1])
def test_zeros_beside_values_of_one_sign(sign, flags):
    for zeros in (1, 20, 400):
        print(sign, flags, zeros, flush=True)
        check([with_zeros(262_144, zeros, sign)], 8, 3, flags=flags)


def test_zeros_in_a_bucket_of_512_cells():
    # 9 M moments, every one kept: the lowest bucket has more than 512 x 64 values; next to no residuals
    check([with_zeros(9_000_000, 100, 1)], 8, 1, alpha=1e6, flags=X.EXCP_FLAG_NO_W2M)


def test_repeated_calls_on_one_context():
    """A context's tables from an earlier, larger call say nothing about the next."""
    ctx = X.Context(400_000, 800_000)
    for n, kind in ((400_000, "both signs"), (150_000, "crowded"), (131_072, "one sign"), (200, "orders"), (399_999, "orders")):
        case = draw(n, n, kind)
        rc, out = gpu_compress(ctx, [case, draw(33, 1, kind)], 0.0, 0.0, 4, 4)
        assert rc == 0 and out[0]["blob"] == O.compress_step(*case, 0.0, 0.0, 4, 4).blob
    ctx.close()
