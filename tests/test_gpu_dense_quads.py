"""The stored layout restored four elements to a lane, at the ends of quads, loads and tiles: 16-bit weights at every
alignment and both widths of a code, byte for byte against the oracle (test_gpu_dense.py has the fp32 weights)."""
import numpy as np
import pytest
import torch

import oracle as O
import paper_2406_11257_amd as X
from test_gpu_dense import code_buffer
from test_gpu_w16 import BF16, F16, bits, case16, compress16, w_to_dev, w_to_host

pytestmark = pytest.mark.gpu
SIZES = [1, 2, 3, 4, 5, 1023, 1024, 1025, 1027, 4095, 4096, 4097, 5122, 8191, 3 * 4096 + 1026]


@pytest.fixture(scope="module")
def ctx():
    c = X.Context(1 << 20, 1 << 20)
    yield c
    c.close()


@pytest.mark.parametrize("flag", [F16, BF16])
@pytest.mark.parametrize("nbits", [3, 4, 7])
@pytest.mark.parametrize("shift", [0, 1, 4])               # elements: 2-, 2- and 8-byte steps from a 16-byte boundary
def test_restored_sixteen_bit_weights_and_moments(ctx, flag, nbits, shift):
    cases = [case16(n, 40 + i, flag) for i, n in enumerate(SIZES)]
    rc, stats, dev = compress16(ctx, cases, flag, nbits=nbits)
    assert rc == 0
    hb = X.excp_head_bytes(nbits)
    export, restore, outs = [], [], []
    for (Wp, *_), st, d in zip(cases, stats, dev):
        n = Wp.size
        codes = [code_buffer(hb)] + [code_buffer(X.excp_dense_bytes(n, nbits)) for _ in range(3)]
        export.append((d[4], int(st.blob_bytes), n, *codes))
        Win = w_to_dev(np.concatenate([np.zeros(shift, Wp.dtype), Wp]), flag)[shift:]
        out = [torch.full((n + shift + 8,), 3.0, dtype=Win.dtype, device="cuda")] + [
            torch.full((n + 8,), 3.0, dtype=torch.float32, device="cuda") for _ in range(2)]
        outs.append(out)
        restore.append((Win, codes[0], hb, n, *codes[1:], out[0][shift:shift + n], out[1][:n], out[2][:n]))
    ctx.excp_export_dense(export)
    assert ctx.excp_collect(check=False)[0] == 0
    ctx.excp_decompress_dense(restore)
    assert ctx.excp_collect(check=False)[0] == 0
    for (Wp, *_), st, d, (Wo, mo, vo) in zip(cases, stats, dev, outs):
        n = Wp.size
        blob = d[4][:int(st.blob_bytes)].cpu().numpy().tobytes()
        W, m, v = O.decompress_step(Wp, blob)
        for got, want in ((w_to_host(Wo[shift:shift + n], flag), W), (mo[:n].cpu().numpy(), m), (vo[:n].cpu().numpy(), v)):
            assert bits(got).tobytes() == bits(want).tobytes()
        for t, at in ((Wo, shift + n), (mo, n), (vo, n)):
            assert bool((t[at:] == 3.0).all()) and bool((Wo[:shift] == 3.0).all()), "written past the tensor"
