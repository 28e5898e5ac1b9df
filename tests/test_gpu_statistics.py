"""The exact median of |W_t - W_prev| and the exact mean of |m| (Sec. 3.2) at the sizes where the passes that
compute them divide their work differently: one workgroup or many per tensor, one or several lists of median
candidates, brackets that hold one value, miss, or overflow.  Everything is compared bit for bit."""
import numpy as np
import pytest
import torch

import oracle as O
import paper_2406_11257_amd as X
from gpu_util import gpu_compress

pytestmark = pytest.mark.gpu
f32 = np.float32


@pytest.fixture(scope="module")
def ctx():
    c = X.Context(1 << 23, 1 << 24)
    yield c
    c.close()


def draw(n, seed, kind):
    g = np.random.default_rng(seed)
    Wp = (g.standard_normal(n) * 0.02).astype(f32)
    d = g.laplace(0, 1e-4, n).astype(f32)
    m = (g.standard_normal(n) * 5e-5).astype(f32)
    if kind == "few values":                       # heavily tied: the bracket collapses, or holds a few values
        d = (g.integers(-3, 4, n) * f32(2.0 ** -14)).astype(f32)
        Wp = (g.integers(-64, 64, n) * f32(2.0 ** -8)).astype(f32)
    elif kind == "half still":                     # the median is zero
        d[g.random(n) < 0.6] = 0.0
    elif kind == "bunched":                        # all values near the median sit in one stretch: its lists overflow
        d = np.sort(d)
    elif kind == "missed":                         # the sampled positions say nothing about the rest
        d[(np.arange(8192, dtype=np.int64) * n) // 8192] = 0.5
        m[::1000] = 3e30
        m[1::1000] = 1e-41
    v = np.full(n, 1e-10, f32)
    return Wp, (Wp + d).astype(f32), m, v


@pytest.mark.parametrize("kind", ["spread", "few values", "half still", "bunched", "missed"])
def test_median_and_mean_are_exact(ctx, kind):
    # around one sub-tile, the sample's size, one workgroup's share, one list, two lists, seven lists
    sizes = [1, 63, 4096, 8191, 8192, 8193, 40961, (1 << 20) - 1, (1 << 21) + 3, 4096 * 2048 - 4095]
    cases = [draw(n, 50 + i, kind) for i, n in enumerate(sizes)]
    print(kind, sizes, flush=True)
    for batch in (cases, cases[::-1], cases[-1:]):         # the shares of the workgroups fall differently
        rc, out = gpu_compress(ctx, batch, nbits=2, iters=0, want_recon=False)
        assert rc == 0
        for (Wp, W, m, _), o in zip(batch, out):
            med = O.lower_median_abs(O.residual(W, Wp))
            total, mean = O.exact_mean_abs(m)
            st = o["stats"]
            assert f32(st.median_abs_dw).tobytes() == f32(med).tobytes()
            assert st.abs_sum_m == total
            assert f32(st.mean_abs_m).tobytes() == f32(mean).tobytes()
            assert f32(st.t_w).tobytes() == f32(f32(5e-5) * f32(med)).tobytes()
            assert f32(st.r_o).tobytes() == f32(f32(2.0) * f32(mean)).tobytes()


def test_non_finite_values_are_counted_wherever_they_are(ctx):
    n = 3_000_001
    Wp, W, m, v = draw(n, 90, "spread")
    small = draw(5000, 91, "spread")
    for pos in (0, 4096 * 700 + 5, n - 1):
        bad = m.copy()
        bad[pos] = np.inf
        rc, out = gpu_compress(ctx, [small, (Wp, W, bad, v), small], nbits=2, iters=0, want_recon=False)
        assert rc == X.EXCP_E_NONFINITE
        assert [o["stats"].nonfinite for o in out] == [0, 1, 0]
