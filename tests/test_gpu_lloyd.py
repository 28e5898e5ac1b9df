"""Lloyd iterations (Sec. 3.3) against the oracle, blob for blob, where the kernels divide the work differently: streams
that one workgroup takes through all iterations and others with a launch per iteration (the line lies at the values that
an iteration is expected to read, and differs with the number of tensors), few and many values in cut buckets, buckets with
one, two and many borders, crowded ones, values of both signs in one bucket, and buckets whose values lie many binary
orders apart."""
import numpy as np
import pytest

import oracle as O
import paper_2406_11257_amd as X
from gpu_util import gpu_compress

pytestmark = pytest.mark.gpu
f32 = np.float32


@pytest.fixture(scope="module")
def ctx():
    c = X.Context(10_000_000, 16_000_000)
    yield c
    c.close()


def draw(n, seed, kind):
    g = np.random.default_rng(seed)
    if kind == "spread":
        d = g.laplace(0, 1e-4, n)
    elif kind == "gap":                     # two signs, nothing near zero: a bucket spans the gap
        d = (1e-4 + g.exponential(3e-5, n)) * g.choice([-1.0, 1.0], n)
    elif kind == "far apart":               # sixty binary orders, both signs: no window holds a bucket's values
        d = 2.0 ** g.uniform(-70, -10, n) * g.choice([-1.0, 1.0], n)
    elif kind == "outliers":                # most centres end up where few values are: many borders in a bucket
        d = np.where(g.random(n) < 0.004, g.uniform(-1, 1, n), g.normal(0, 1e-6, n))
    else:                                   # "tied": a few values and strays beside them
        d = g.integers(-4, 5, n) * 2.0 ** -14 + np.where(g.random(n) < 0.01, g.normal(0, 1e-5, n), 0.0)
    m = d[::-1] * 0.5
    v = m * m * np.exp(g.normal(0, 1, n)) + 1e-16
    return np.zeros(n, f32), d.astype(f32), m.astype(f32), v.astype(f32)


def check(ctx, cases, nbits, iters, alpha=0.0, beta=0.0):
    rc, out = gpu_compress(ctx, cases, alpha, beta, nbits, iters)
    assert rc == 0
    for (Wp, W, m, v), o in zip(cases, out):
        ref = O.compress_step(Wp, W, m, v, alpha, beta, nbits, iters)
        assert o["stats"].n_w == ref.n_w and o["stats"].n_o == ref.n_o
        assert o["blob"] == ref.blob


@pytest.mark.parametrize("kind", ["spread", "gap", "far apart", "outliers", "tied"])
def test_every_way_through_an_iteration(ctx, kind):
    for nbits, sizes in ((8, [255, 5000, 60_001, 528_416, 528_417]), (2, [3, 4096, 300_003]), (4, [16, 9000, 400_001])):
        for iters in (1, 10):
            print(kind, nbits, iters, sizes, flush=True)
            check(ctx, [draw(n, 7 * nbits + i, kind) for i, n in enumerate(sizes)], nbits, iters)


@pytest.mark.parametrize("kind", ["outliers"])
def test_a_launch_per_iteration_with_fifteen_centres(ctx, kind):
    check(ctx, [draw(9_586_981, 5, kind), draw(1000, 6, kind)], 4, 2)


def test_no_iterations_and_the_usual_thresholds(ctx):
    check(ctx, [draw(n, n, "spread") for n in (1, 700, 600_000)], 8, 0, alpha=5e-5, beta=2.0)
    check(ctx, [draw(n, n, "spread") for n in (1, 700, 600_000)], 8, 10, alpha=5e-5, beta=2.0)


def skewed(n, seed, kind):
    """Residuals and moments that the value -> bucket map cannot spread: nearly all in one bucket, most centres with them."""
    g = np.random.default_rng(seed)
    sign = g.choice([-1.0, 1.0], n)
    if kind == "sign step":                 # +-lr as fp32 weights round it, and a few smaller steps
        Wp = (g.standard_normal(n) * 0.02).astype(f32)
        d = sign * 1e-4 * np.where(g.random(n) < 0.02, g.random(n), 1.0)
    else:                                   # "bunched": one thirtieth of an octave, a few values far away
        Wp = np.zeros(n, f32)
        d = sign * np.where(g.random(n) < 0.002, 2.0 ** (-40 * g.random(n) - 13), (1 + 0.02 * g.random(n)) * 2.0 ** -13)
    W = (Wp + d).astype(f32)
    m = (d * 0.1).astype(f32)
    return Wp, W, m, (m.astype(np.float64) ** 2 * np.exp(g.normal(0, 1, n)) + 1e-16).astype(f32)


@pytest.mark.parametrize("kind", ["sign step", "bunched"])
def test_crowded_buckets_on_both_sides_of_the_lines(ctx, kind):
    # one workgroup a stream up to 2^17 elements (2^24 / 254 in 8 bits, 2^22 in 2); beyond, the filled buckets decide
    for nbits, sizes in ((4, [131_072, 5]), (4, [131_073, 3000, 7]), (4, [700_001]), (8, [66_052]), (8, [66_053, 400]), (2, [300_000]), (2, [4_194_305]), (6, [200_001])):
        print(kind, nbits, sizes, flush=True)
        check(ctx, [skewed(n, n + nbits, kind) for n in sizes], nbits, 3)


@pytest.mark.parametrize("nbits, n", [(2, 4_200_001), (3, 1_200_001), (4, 460_001), (5, 210_001), (6, 300_001), (7, 140_001), (8, 70_001)])
def test_even_buckets_of_one_tensor_in_both_ways(ctx, nbits, n):
    # (by one workgroup a stream: at the usual thresholds, or because the larger buckets have cells)
    check(ctx, [draw(n, nbits, "spread")], nbits, 2)
    check(ctx, [draw(n, nbits, "spread"), draw(100, 3, "spread")], nbits, 2, alpha=5e-5, beta=2.0)


@pytest.mark.parametrize("nbits", [3, 5, 8])
def test_even_buckets_shared_out(ctx, nbits):
    # everything kept and known beforehand to be more than cells are made for
    check(ctx, [draw(1_700_001, nbits, "spread")], nbits, 2)


def test_both_ways_in_one_group(ctx):
    # more streams than compute units: tensors go either way by themselves
    sizes = [140_001, 700, 100_003, 1, 140_002] + [300 + 7 * i for i in range(90)]
    check(ctx, [draw(n, n, "spread") for n in sizes], 8, 2)
    check(ctx, [skewed(n, n, "bunched") if i < 3 else draw(n, n, "gap") for i, n in enumerate(sizes)], 8, 2)


def test_more_large_tensors_of_wide_codes_than_accumulators():
    # 341 tensors of 255 centres have accumulators; smaller ones do without, and cost no group of their own
    ctx = X.Context(70_000, 27_000_000)
    small, large = [draw(n, n, "spread") for n in (2000, 3001)], draw(66_100, 1, "spread")
    ctx.excp_set_profiling(True)
    try:
        for cases, groups in (([small[i & 1] for i in range(700)], 1), ([large] * 120 + [small[0]] * 600, 1), ([large] * 341 + [small[0]], 1),
                              ([small[1]] + [large] * 342, 2)):
            rc, out = gpu_compress(ctx, cases, 0.0, 0.0, 8, 1, want_recon=False)
            assert rc == 0 and ctx.stage_times()["layout"][1] == groups
            for i in (0, len(cases) // 2, len(cases) - 1):
                assert out[i]["blob"] == O.compress_step(*cases[i], 0.0, 0.0, 8, 1).blob
    finally:
        ctx.close()


def test_crowded_buckets_cost_no_multiple_of_even_ones(ctx):
    # (one workgroup for all of a million bunched values took 55 times as long as for even ones)
    ctx.excp_set_profiling(True)
    try:
        ms = {}
        for kind in ("even", "sign step", "bunched"):
            case = draw(1_000_003, 4, "spread") if kind == "even" else skewed(1_000_003, 4, kind)
            for _ in range(3):
                gpu_compress(ctx, [case], 0.0, 0.0, 4, 10, want_recon=False)
                ms[kind] = min(ms.get(kind, 1e9), ctx.stage_times()["km_iter"][0])
        assert max(ms.values()) < 10 * ms["even"], ms
    finally:
        ctx.excp_set_profiling(False)
