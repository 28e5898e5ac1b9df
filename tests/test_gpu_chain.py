"""Chains of checkpoints (Alg. 3) where the one-pass kernel divides its work: quarters of 1024 elements, tiles of 4096,
tensors of several tiles, every element kept (more code words than a wave loads at once) and few, and codebooks
larger than a wave."""
import numpy as np
import pytest
import torch

import oracle as O
import paper_2406_11257_amd as X
from gpu_util import to_dev

pytestmark = pytest.mark.gpu
f32 = np.float32
SIZES = [1, 63, 1024, 1025, 3 * 1024 + 17, 4095, 4096, 4097, 9 * 4096 + 1, 17 * 4096]


@pytest.mark.parametrize("flags", [0, X.EXCP_FLAG_W_F16, X.EXCP_FLAG_W_BF16])
@pytest.mark.parametrize("alpha, widths", [(0.0, (8, 2, 7)), (5e-5, (4, 8)), (3e-4, (4,))])
def test_quarters_tiles_and_code_widths(alpha, widths, flags):
    ctx = X.Context(max(SIZES), sum(SIZES))
    chains, dev, outs = [], [], []
    for n in SIZES:
        g = np.random.default_rng(n)
        W0 = O.narrow((g.standard_normal(n) * 0.02).astype(f32), flags)
        W, hat, blobs = O.widen(W0, flags), W0, []
        for nbits in widths:
            W = (W + g.laplace(0, 1e-4 if flags == 0 else 3e-3, n)).astype(f32)
            m = (g.standard_normal(n) * 5e-5).astype(f32)
            v = (m.astype(np.float64) ** 2 * g.lognormal(0, 1, n) + 1e-16).astype(f32)
            r = O.compress_step(hat, O.narrow(W, flags), m, v, alpha, 2.0, nbits, 2, flags=flags)
            blobs.append(r.blob)
            hat = r.W_recon
        chains.append((W0, blobs))
        stored = torch.from_numpy(np.ascontiguousarray(W0).view(f32 if flags == 0 else np.int16)).cuda()
        wo = torch.zeros_like(stored)
        outs.append(wo)
        dev.append((stored, [torch.from_numpy(np.frombuffer(b, np.uint8).copy()).cuda() for b in blobs],
                    [len(b) for b in blobs], wo, None, None))
    if flags:
        view = torch.float16 if flags == X.EXCP_FLAG_W_F16 else torch.bfloat16
        dev = [(d[0].view(view), *d[1:3], d[3].view(view), None, None) for d in dev]
    print(alpha, widths, flags, flush=True)
    ctx.excp_reconstruct_chain(dev)
    rc, stats = ctx.excp_collect(check=False)
    assert rc == 0
    for (W0, blobs), wo in zip(chains, outs):
        ref = O.reconstruct_chain(W0, blobs)[0]
        assert wo.cpu().numpy().tobytes() == np.ascontiguousarray(ref).tobytes()
    ctx.close()
