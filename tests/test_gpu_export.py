"""The export of the stored layout at the edges of what a lane (16 elements), a quarter of a tile (1024) and a wave (4096)
take, for every code width, with few and with all elements kept (more words of codes than a wave loads at once), and with
M_o bits per kept residual and per element, with a tile to a workgroup (16 of them) and to a wave (1120): the blobs are the oracle's, and so are the codes, byte for byte."""
import numpy as np
import pytest
import torch

import oracle as O
import paper_2406_11257_amd as X
from test_gpu_dense import CANARY, code_buffer
from test_gpu_parity import case

pytestmark = pytest.mark.gpu
SIZES = [1, 2, 15, 16, 17, 1023, 1024, 1025, 1040, 4095, 4096, 4097, 2 * 4096 + 3 * 1024 + 7]


@pytest.mark.parametrize("nbits", [2, 3, 4, 5, 6, 7, 8])
@pytest.mark.parametrize("flags", [0, X.EXCP_FLAG_NO_W2M])
@pytest.mark.parametrize("alpha, beta", [(0.0, 0.0), (5e-5, 2.0)])
@pytest.mark.parametrize("copies", [1, 70])
def test_codes_of_every_element(nbits, flags, alpha, beta, copies):
    blobs = [O.compress_step(*case(n, 60 + i), alpha, beta, nbits, 2, flags=flags).blob for i, n in enumerate(SIZES)]
    on_gpu = [torch.from_numpy(np.frombuffer(b, np.uint8).copy()).cuda() for b in blobs]
    items, bufs = [], []
    for _ in range(copies):
        for n, t in zip(SIZES, on_gpu):
            bufs.append([code_buffer(X.excp_dense_bytes(n, nbits)) for _ in range(3)])
            items.append((t, t.numel(), n, None, *bufs[-1]))
    ctx = X.Context(max(SIZES), copies * sum(SIZES))
    ctx.excp_export_dense(items)
    rc, _ = ctx.excp_collect(check=False)
    ctx.close()
    assert rc == 0
    wanted = [O.export_dense(b)[1:] for b in blobs]
    for i, got in enumerate(bufs):
        n = SIZES[i % len(SIZES)]
        for t, want in zip(got, wanted[i % len(SIZES)]):
            a = t.cpu().numpy()
            size = X.excp_dense_bytes(n, nbits)
            assert a[:size].tobytes() == want.tobytes() and bool((a[size:] == CANARY).all()), n
