"""Bucket totals and initial centres against the oracle, blob for blob, in each form that a group's size and its weights'
storage choose: a bucket or four to a workgroup (the line lies at 1024 sets of four, that is at six tensors on 256 compute
units), small buckets side by side and large ones shared, and the counted repetitions of tied data."""
import numpy as np
import pytest
import torch

import oracle as O
import paper_2406_11257_amd as X

pytestmark = pytest.mark.gpu
f32 = np.float32


def draw(n, flags, tied):
    g = np.random.default_rng(n)
    Wp = O.narrow((g.standard_normal(n) * 0.02).astype(f32), flags)
    step = g.integers(-3, 4, n) * 2.0 ** -11 + np.where(g.random(n) < 0.02, g.normal(0, 1e-3, n), 0.0) if tied else g.laplace(0, 1e-3, n)
    W = O.narrow((O.widen(Wp, flags) + step).astype(f32), flags)
    m = (g.standard_normal(n) * 5e-5).astype(f32)
    v = (m.astype(np.float64) ** 2 * g.lognormal(0, 1, n) + 1e-16).astype(f32)
    return Wp, W, m, v


@pytest.mark.parametrize("tied", [False, True])
@pytest.mark.parametrize("flags", [0, X.EXCP_FLAG_W_F16, X.EXCP_FLAG_W_BF16])
@pytest.mark.parametrize("sizes", [[300_001, 1000], [700_003, 3, 4097, 255, 70_000, 2048, 1025, 12_289]])
def test_every_form_of_the_totals(sizes, flags, tied):
    ctx = X.Context(max(sizes), sum(sizes))
    kind = {0: torch.float32, X.EXCP_FLAG_W_F16: torch.float16, X.EXCP_FLAG_W_BF16: torch.bfloat16}[flags]
    put = lambda a: torch.from_numpy(np.ascontiguousarray(a).view(f32 if flags == 0 else np.int16)).cuda().view(kind)
    cases = [draw(n, flags, tied) for n in sizes]
    for nbits, alpha in ((4, 0.0), (8, 5e-5)):
        blobs = [torch.zeros(X.excp_blob_bound(n, nbits), dtype=torch.uint8, device="cuda") for n in sizes]
        print(sizes, flags, tied, nbits, flush=True)
        ctx.excp_compress_tensors([(put(Wp), put(W), torch.from_numpy(m).cuda(), torch.from_numpy(v).cuda(), b, None)
                                   for (Wp, W, m, v), b in zip(cases, blobs)], alpha, 2.0, nbits, 3, flags)
        rc, stats = ctx.excp_collect(check=False)
        assert rc == 0
        for c, b, st in zip(cases, blobs, stats):
            assert b[:st.blob_bytes].cpu().numpy().tobytes() == O.compress_step(*c, alpha, 2.0, nbits, 3, flags=flags).blob
    ctx.close()
