"""Lloyd iterations (Sec. 3.3) against the oracle, blob for blob, where the kernels divide the work differently: streams
that one workgroup takes through all iterations and larger ones with a launch per iteration (the line lies at
n (K - 1) = 2^27 for a tensor of n values and K centres), few and many values in cut buckets, buckets with one, two and
many borders, values of both signs in one bucket, and buckets whose values lie many binary orders apart."""
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
